// Standard attention layer that also emits the shared scores (Sec. 2.1 Eq. 1-2), bf16 on MFMA.
//
// One workgroup = one head and 128 consecutive query rows, one wave per block of 32 rows,
// streaming over 32-key tiles up to the diagonal.  The K tile (and the V tile) of a step is
// loaded once per workgroup into LDS (double buffered, one barrier per tile) and read by the
// four waves as MFMA operands: a fourth of the global loads of a wave-private stream.
// Both products use the 32x32x16 MFMA and keep the query row on the lane index
// (lane = 32 half + r), so the softmax statistics and the probabilities never change lanes:
//   scores  D[key, row] = sum_t K[key,t] Q[row,t]   A = K rows, B = Q^T (8 operands, resident).
//           MFMA row m is given key 16 (m/16) + 8 ((m/4)%2) + 4 ((m/8)%2) + m%4 so that lane
//           (r, half) ends with keys 8 half .. 8 half + 7 and 16 + 8 half .. 16 + 8 half + 7:
//           two 16-byte half stores.
//   output  D[d, row] = sum_key V^T[d,key] P^T[key,row]   A = V^T, whose columns the transposing LDS read hands out
//           of the V rows as they are, B = the lane's probabilities as they are.
// A = Q K^T * scale is stored as half; the softmax works on the float32 values.
// A workgroup takes one row group, long ones first (tests can make it take the x-th longest and the x-th shortest).  Where
// there are few workgroups it has a second set of four waves, and each set takes half of the keys (NH, std_key_halves()).
#pragma once
#include "kernels_prefill.h"

namespace lisa {

typedef float f32x16 __attribute__((ext_vector_type(16)));

struct StdPrefillArgs {
  const bf16_t* q;        // [B,H,Lq,128]
  const bf16_t* k;        // [B,Hkv,Lk,128]
  const bf16_t* v;        // [B,Hkv,Lk,128] or null (scores only)
  half_t* scores;         // [B,H,Lq,Lk] or null
  const void* given;      // GIVEN mode: scores [B,H,Lq,Lk] to take instead of Q K^T (then q, k unused):
                          // float32 (GIVEN = 1) or IEEE half (GIVEN = 2)
  void* out;              // [B,Lq,H,128] or null
  int H, Hkv, Lq, Lk, causal, out_f32;
  int pair;               // 1: a workgroup takes two row groups (ceil(n_groups / 2) slots), 0: one
  int by_length;          // grid (H, B, slots), else (H, slots, B)
  float scale;
};

__device__ __forceinline__ float halves_max(float v) {
  const unsigned u = __float_as_uint(v);
  auto q = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
__device__ __forceinline__ float halves_sum(float v) {
  const unsigned u = __float_as_uint(v);
  auto q = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

constexpr int SP_ROWS = 32;                 // rows per wave
constexpr int SP_WAVES = 4;
constexpr int SP_GROUP = SP_ROWS * SP_WAVES;   // rows per workgroup pass
constexpr int SP_TK = 32;
constexpr int SP_KROW = 128 * 2 + 16;       // bytes per key row of the K tile in LDS (padded: no bank conflicts)
constexpr int SP_KTILE = SP_TK * SP_KROW;   // 8704
constexpr int SP_VROW = 128 * 2 + 32;       // bytes per key row of the V tile in LDS: the four rows that 16 lanes of a
                                            // transposing read touch fall into different banks
constexpr int SP_VTILE = SP_TK * SP_VROW;   // 9216
constexpr int SP_SROW = 2 * SP_TK * 2 + 16;  // bytes per row of a wave's score staging tile (64 keys, padded)
constexpr int SP_STILE = SP_ROWS * SP_SROW;  // 4608

// An operand of eight keys from rows of SP_VROW bytes: keys 0 .. 3 and 4 .. 7 of the lane's address (see k_std_prefill).
__device__ __forceinline__ bf16x8 read_columns(const unsigned char* p) {
  typedef s16x4 __attribute__((address_space(3))) lds_s16x4;
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * SP_VROW));
  return __builtin_bit_cast(bf16x8, (s16x8){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
}

constexpr int SP_OROW = 128 + 4;            // floats per row of a partial result
// LDS bytes of one key half: two K tiles, the four staging tiles, two V tiles.
constexpr int std_prefill_head_lds(bool with_v) {
  return 2 * SP_KTILE + SP_WAVES * SP_STILE + (with_v ? 2 * SP_VTILE : 0);
}

// grid (H, pair ? ceil(n_groups / 2) : n_groups, B) with n_groups = ceil(Lq / 128), block 256 NH.  The head is the
// fastest grid index: consecutive workgroups go to different XCDs, so an XCD works on every
// eighth head and its L2 fetches the K / V of those heads only (they are what every row group
// of a head re-reads).
// Requires d_k = 128, Lk % 8 == 0 of row-major scores (tiled ones: any Lk >= 8).
// GIVEN: the scores are read from a.given (the A_n that a LiSA scores kernel left there) instead
// of being computed; the rest (masking, online softmax, P V) is the same.
// TILED: scores are written (GIVEN = 2: read) as [B,ceil(Lq/16),ceil(Lk/32),H,16,32].
// V is staged as it lies in memory (a launch that regrouped it by key chunks before was 8 - 11 us of a layer of 2048 tokens).
// NH = 2: eight waves, two per row block, which take the even and the odd key tiles, each half with buffers of its own, and
// merge their softmax states at the end: half the chain of tiles where there
// are too few workgroups to hide it (std_key_halves).
template <bool WITH_V, int GIVEN = 0, bool TILED = false, int NH = 1>
__global__ __launch_bounds__(256 * NH, 2) void k_std_prefill(StdPrefillArgs a) {
  constexpr int DK = 128;
  __shared__ __align__(16) unsigned char lds[NH * std_prefill_head_lds(WITH_V)];
  const int tid = threadIdx.x & 255, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);                               // row block of the wave
  const int kh = NH == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);    // its key half
  unsigned char* ks_ = lds + kh * (2 * SP_KTILE);
  unsigned char* ss_ = lds + NH * (2 * SP_KTILE);       // score staging, one tile per wave
  unsigned char* vs_ = ss_ + NH * (SP_WAVES * SP_STILE) + kh * (2 * SP_VTILE);
  const int r = lane & 31, half = lane >> 5;
  const int b = a.by_length ? blockIdx.y : blockIdx.z, h = blockIdx.x, slot = a.by_length ? blockIdx.z : blockIdx.y;
  const int Lq = a.Lq, Lk = a.Lk, H = a.H;
  const int shift = Lk - Lq;
  const int kv = h / (H / a.Hkv);
  const float LOG2E = 1.4426950408889634f;
  const int n_groups = (Lq + SP_GROUP - 1) / SP_GROUP;
  // key of MFMA row m = r (see the header)
  const int key_of_r = 16 * (r >> 4) + 8 * ((r >> 2) & 1) + 4 * ((r >> 3) & 1) + (r & 3);
  const bf16_t* kbase = GIVEN ? nullptr : a.k + ((size_t)b * a.Hkv + kv) * Lk * DK;
  const bf16_t* vbase = WITH_V ? a.v + ((size_t)b * a.Hkv + kv) * Lk * DK : nullptr;
  // cooperative tile loads: thread -> two 16-byte chunks (key, 8 features) of the K and of the V tile
  const int ck_key = tid >> 4, ck_c = tid & 15;          // chunk u: key ck_key + 16 u
  // operand addresses in LDS
  const int k_rd = key_of_r * SP_KROW + half * 16;       // + 32 ks
  // transposing read: lane s of a 16-lane group passes the address of key s / 4, features 4 (s % 4) .. and receives
  // feature s of keys 0 .. 3; lanes 16 .. 31 of a half take the next 16 features.  + 16 s SP_VROW + 64 db
  const int v_rd = (8 * half + ((lane & 15) >> 2)) * SP_VROW + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;

  for (int rep = 0; rep < 2; ++rep) {
    const int grp = rep ? slot : n_groups - 1 - slot;
    if (rep && (!a.pair || grp >= n_groups - 1 - grp)) break;   // (the middle group of an odd count is alone)
    const int i0 = grp * SP_GROUP + wv * SP_ROWS;          // first row of this wave
    const bool have_rows = i0 < Lq;
    const int my_row = min(i0 + r, Lq - 1);
    const int vis_row = a.causal ? min(Lk, my_row + 1 + shift) : Lk;
    const int i_last_w = min(i0 + SP_ROWS - 1, Lq - 1);
    const int n_tiles_w =
        have_rows ? ((a.causal ? min(Lk, i_last_w + 1 + shift) : Lk) + SP_TK - 1) / SP_TK : 0;
    const int i_last_g = min(grp * SP_GROUP + SP_GROUP - 1, Lq - 1);
    const int n_tiles = ((a.causal ? min(Lk, i_last_g + 1 + shift) : Lk) + SP_TK - 1) / SP_TK;
    const int n_full =
        (have_rows && i0 + SP_ROWS <= Lq) ? (a.causal ? min(Lk, i0 + 1 + shift) : Lk) / SP_TK : 0;

    // B operands of the score product: Q[row][16 ks + 8 half + e]
    bf16x8 qop[DK / 16];
    if (!GIVEN) {
      const bf16_t* qp = a.q + (((size_t)b * H + h) * Lq + my_row) * DK + 8 * half;
#pragma unroll
      for (int ks = 0; ks < DK / 16; ++ks) qop[ks] = *(const bf16x8*)(qp + 16 * ks);
    }
    const size_t grow_at = (((size_t)b * H + h) * Lq + my_row) * Lk;
    const float* grow = GIVEN == 1 ? (const float*)a.given + grow_at : nullptr;
    const half_t* grow_h = GIVEN == 2 ? (const half_t*)a.given + grow_at : nullptr;
    const int n_kt = (Lk + SP_TK - 1) / SP_TK;               // tile grid of the tiled score layout
    // (tiled: the H pieces of a tile follow each other, 1 KB each; see k_lisa_prefill_fused)
    const size_t seq_elems = TILED ? (size_t)((Lq + 15) / 16) * n_kt * H * (16 * SP_TK) : (size_t)H * Lq * Lk;
    half_t* sbase = a.scores ? a.scores + (size_t)b * seq_elems + (size_t)h * (TILED ? (size_t)16 * SP_TK : (size_t)Lq * Lk)
                             : nullptr;
    unsigned char* stg = ss_ + (kh * SP_WAVES + wv) * SP_STILE;

    // The K / V tile of a step travels through registers: loaded three tiles ahead into one of two
    // register sets, written to LDS one tile ahead.  Two sets rather than one because loads and
    // stores complete in one order behind one counter, and the score stores below are conditional
    // (uncountable for the compiler): with one set the wait for the tile loads at the top of a step
    // was a wait for everything, the score stores of the step before included; with two the loads
    // of the other set lie between, and only what is older than those has to be complete.
    typedef pf_u32x4 TileRegs[2][2];                       // [K, V][chunk]
    TileRegs regs_a, regs_b;
    auto load_tile = [&](int tile, TileRegs& tr) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int j = min(tile * SP_TK + ck_key + 16 * u, Lk - 1);
        if (!GIVEN) tr[0][u] = *(const pf_u32x4*)(kbase + (size_t)j * DK + 8 * ck_c);
        if (WITH_V) tr[1][u] = *(const pf_u32x4*)(vbase + (size_t)j * DK + 8 * ck_c);
      }
    };
    auto store_tile = [&](int buf, const TileRegs& tr) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (!GIVEN) *(pf_u32x4*)(ks_ + buf * SP_KTILE + (ck_key + 16 * u) * SP_KROW + ck_c * 16) = tr[0][u];
        if (WITH_V) *(pf_u32x4*)(vs_ + buf * SP_VTILE + (ck_key + 16 * u) * SP_VROW + ck_c * 16) = tr[1][u];
      }
    };
    // GIVEN = 2: the wave's scores of a tile are loaded two tiles ahead (nothing else hides the
    // latency of these loads: there is no score product to wait behind)
    f16x8 gq[2][2];
    // (tiled: row my_row of head h, tile t at (((my_row / 16) n_kt + t) H + h) KB + 64 (my_row % 16) bytes)
    const half_t* grow_t = GIVEN == 2 ? (const half_t*)a.given + (size_t)b * seq_elems +
                                            ((size_t)(my_row >> 4) * n_kt * H + h) * (16 * SP_TK) +
                                            (my_row & 15) * SP_TK + 8 * half
                                      : nullptr;
    auto load_scores = [&](int tile, f16x8 (&dst)[2]) {
#pragma unroll
      for (int u = 0; u < 2; ++u)    // (keys beyond Lk: any in-bounds 8 scores will do, those positions are masked)
        dst[u] = *(const f16x8*)(TILED ? grow_t + (size_t)tile * H * (16 * SP_TK) + 16 * u
                                         : grow_h + min(tile * SP_TK + 16 * u + 8 * half, Lk - 8));
    };
    if (rep) __syncthreads();                              // the first pass is done with both buffers
    const int n_steps = (n_tiles + NH - 1) / NH;
    auto tile_of = [&](int st) { return min(NH * st + kh, n_tiles - 1); };
    load_tile(tile_of(0), regs_a);
    store_tile(0, regs_a);
    load_tile(tile_of(1), regs_a);                         // set a: odd steps, set b: even steps
    load_tile(tile_of(2), regs_b);
    if (GIVEN == 2) {
      load_scores(tile_of(0), gq[0]);
      load_scores(tile_of(1), gq[1]);
    }

    f32x16 o[DK / 32];
#pragma unroll
    for (int db = 0; db < DK / 32; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    // Row-major scores leave in whole 128-byte pieces of a row (64 keys = the tiles t and t + 1 of the pair that `tile`
    // belongs to; 64-byte pieces reach HBM at about half the rate): `n` pieces of 8 rows each from row 8 u0 on.
    auto flush_rows = [&](int tile, const unsigned char* from, int u0, int n) {
      const int jc = (tile >> 1) * (2 * SP_TK) + 8 * (lane & 7);
      const bool pair_full = (tile | 1) < n_full;
#pragma unroll
      for (int u = 0; u < n; ++u) {
        const int row = 8 * (u0 + u) + (lane >> 3), gi = i0 + row;
        const f16x8 hv = *(const f16x8*)(from + row * SP_SROW + (lane & 7) * 16);
        const int vis = gi < Lq ? (a.causal ? min(Lk, gi + 1 + shift) : Lk) : 0;
        half_t* sp = sbase + (size_t)min(gi, Lq - 1) * Lk + jc;
        if (pair_full || jc + 8 <= vis) {
          __builtin_nontemporal_store(__builtin_bit_cast(pf_u32x4, hv), (pf_u32x4*)sp);
        } else if (jc < vis) {
          int rel = vis - jc;                              // (kept inside this branch: registers)
          asm volatile("" : "+v"(rel));
          store_row_part(sp, __builtin_bit_cast(pf_u32x4, hv), rel);
        }
      }
    };
    // NH = 2, row-major: the pair is made by both halves and leaves behind the next barrier, half of the rows each
    auto flush_pair = [&](int st) {
      if (!TILED && NH == 2 && !GIVEN && a.scores && st >= 0 && NH * st < n_tiles_w)
        flush_rows(NH * st, ss_ + ((st & 1) * SP_WAVES + wv) * SP_STILE, 2 * kh, 2);
    };
    auto step = [&](int st, TileRegs& tr) {                // tr holds the tile of step st + 1
      const int tile = NH * st + kh;
      // the tile is complete in buffer st & 1, and every wave is done with the other buffer
      lds_barrier();
      store_tile((st + 1) & 1, tr);
      load_tile(tile_of(st + 3), tr);
      flush_pair(st - 1);
      if (tile >= n_tiles_w) return;                       // beyond this wave's diagonal (wave-uniform)
      const unsigned char* kt = ks_ + (st & 1) * SP_KTILE;
      const unsigned char* vtl = vs_ + (st & 1) * SP_VTILE;
      const int j0 = tile * SP_TK;
      // an[8 u + e] = score of key j0 + 16 u + 8 half + e for row r
      float an[16];
      if (GIVEN == 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
          for (int e = 0; e < 8; ++e) an[8 * u + e] = (float)gq[0][u][e];
          gq[0][u] = gq[1][u];
        }
        load_scores(tile_of(st + 2), gq[1]);
      } else if (GIVEN == 1) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const float* gp = grow + min(j0 + 16 * u + 8 * half, Lk - 8);
          const float4 lo = *(const float4*)gp, hi = *(const float4*)(gp + 4);
          an[8 * u + 0] = lo.x, an[8 * u + 1] = lo.y, an[8 * u + 2] = lo.z, an[8 * u + 3] = lo.w;
          an[8 * u + 4] = hi.x, an[8 * u + 5] = hi.y, an[8 * u + 6] = hi.z, an[8 * u + 7] = hi.w;
        }
      } else {
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
        for (int ks = 0; ks < DK / 16; ++ks) {
          const bf16x8 kop = *(const bf16x8*)(kt + k_rd + 32 * ks);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kop, qop[ks], acc, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) an[v] = acc[v] * a.scale;
      }
      const bool full = tile < n_full;
      const int jl = j0 + 8 * half;
      if (a.scores) {
        // A leaves through a staging tile
        f16x8 hv0, hv1;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          hv0[e] = f32_to_half_sat(an[e]);
          hv1[e] = f32_to_half_sat(an[8 + e]);
        }
        unsigned char* sl = (!TILED && NH == 2 ? ss_ + ((st & 1) * SP_WAVES + wv) * SP_STILE : stg) + r * SP_SROW + (tile & 1) * 64 + 16 * half;
        *(f16x8*)sl = hv0;
        *(f16x8*)(sl + 32) = hv1;
        if (TILED) {
          // tiled layout: the wave's 32 rows are two row blocks, one 1 KB tile each per step
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int rbq = (i0 >> 4) + q;
            if (16 * rbq >= Lq) continue;                      // (wave-uniform)
            const f16x8 hv =
                *(const f16x8*)(stg + (16 * q + (lane >> 2)) * SP_SROW + (tile & 1) * 64 + (lane & 3) * 16);
            // (non-temporal: nobody reads the scores before the whole tensor is written; 2.45 -> 2.14 ms
            // on the LLaMA3-8B shape, and the layer that reads them next is not slower, also where
            // the tensor would fit the last-level cache)
            __builtin_nontemporal_store(__builtin_bit_cast(pf_u32x4, hv),
                                        (pf_u32x4*)((char*)sbase + ((size_t)rbq * n_kt + tile) * H * (16 * SP_TK * 2) + lane * 16));
          }
        } else if (NH == 1 && ((tile & 1) == 1 || tile == n_tiles_w - 1)) {
          flush_rows(tile, stg, 0, 4);
        }
      }
      if (WITH_V) {
        // (TILED has the registers for it: the operands of P V are read ahead of the softmax)
        bf16x8 vop[2][DK / 32];
        auto read_v = [&]() {
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int db = 0; db < DK / 32; ++db) vop[s][db] = read_columns(vtl + v_rd + 16 * s * SP_VROW + 64 * db);
        };
        if (TILED) {
          read_v();
          __builtin_amdgcn_sched_barrier(0);
        }
        if (!full) {
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (jl + 16 * (v >> 3) + (v & 7) >= vis_row) an[v] = -INFINITY;
        }
        float mx = max2_raw(an[0], an[15]);
#pragma unroll
        for (int v = 1; v < 15; v += 2) mx = max3_raw(mx, an[v], an[v + 1]);
        mx = halves_max(mx);
        const float m_new = fmaxf(m_run, mx);
        // (no key seen yet, every p is 0: given scores may be -inf, masked, and a half may start beyond a row's diagonal)
        const float m2 = (GIVEN || NH == 2) && m_new == -INFINITY ? 0.f : m_new * LOG2E;
        const float alpha = fast_exp2(m_run * LOG2E - m2);
        m_run = m_new;
        float ps = 0.f;
        bf16x8 pop[2];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float p = fast_exp2(__builtin_fmaf(an[v], LOG2E, -m2));
          ps += p;
          pop[v >> 3][v & 7] = (__bf16)p;
        }
        l_run = l_run * alpha + ps;
        if (__any(alpha != 1.f)) {
#pragma unroll
          for (int db = 0; db < DK / 32; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[db][v] *= alpha;
        }
        if (!TILED) read_v();
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int db = 0; db < DK / 32; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[s][db], pop[s], o[db], 0, 0, 0);
      }
    };
    // (everything loaded so far has arrived before the loop is entered: the wait counts inside the
    // loop then follow from the loop's own issue order, not from that of the prologue)
    __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0), others untouched
    int st = 0;
    for (; st + 1 < n_steps; st += 2) {                    // (both steps on every path round the loop)
      step(st, regs_a);
      step(st + 1, regs_b);
    }
    if (st < n_steps) step(st, regs_a);
    if constexpr (!TILED && NH == 2 && !GIVEN) {
      lds_barrier();
      flush_pair(n_steps - 1);
    }

    if constexpr (WITH_V && NH == 2) {
      // the odd half leaves its state in the LDS, the even one goes on with both
      float* o_s = (float*)lds + wv * (SP_ROWS * SP_OROW);
      float* ml_s = (float*)lds + SP_WAVES * SP_ROWS * SP_OROW + wv * (2 * SP_ROWS);
      __syncthreads();
      if (kh == 1) {
        const float l1 = halves_sum(l_run);
        if (half == 0) *(float2*)(ml_s + 2 * r) = make_float2(m_run, l1);
#pragma unroll
        for (int db = 0; db < DK / 32; ++db)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4)
            *(float4*)(o_s + r * SP_OROW + 32 * db + 8 * q4 + 4 * half) =
                make_float4(o[db][4 * q4], o[db][4 * q4 + 1], o[db][4 * q4 + 2], o[db][4 * q4 + 3]);
      }
      __syncthreads();
      if (kh == 1) return;
      const float2 ml = *(const float2*)(ml_s + 2 * r);
      const float M = fmaxf(m_run, ml.x), M2 = M == -INFINITY ? 0.f : M * LOG2E;
      const float f0 = fast_exp2(m_run * LOG2E - M2), f1 = fast_exp2(ml.x * LOG2E - M2);
      // (l_run is this lane's share of the row's sum, ml.y the other half's whole: half of it to each of the two lanes)
      l_run = l_run * f0 + 0.5f * ml.y * f1;
#pragma unroll
      for (int db = 0; db < DK / 32; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const float4 x = *(const float4*)(o_s + r * SP_OROW + 32 * db + 8 * q4 + 4 * half);
          o[db][4 * q4] = o[db][4 * q4] * f0 + x.x * f1;
          o[db][4 * q4 + 1] = o[db][4 * q4 + 1] * f0 + x.y * f1;
          o[db][4 * q4 + 2] = o[db][4 * q4 + 2] * f0 + x.z * f1;
          o[db][4 * q4 + 3] = o[db][4 * q4 + 3] * f0 + x.w * f1;
        }
    }
    if (WITH_V) {
      // O[row][h][32 db + 8 (v/4) + 4 half + v%4] = o[db][v] / l
      const float l = halves_sum(l_run);
      const float inv = GIVEN && l == 0.f ? 0.f : 1.f / l;   // (a row that sees nothing gives zeros)
      if (i0 + r < Lq) {
        const size_t at = (((size_t)b * Lq + i0 + r) * H + h) * DK + 4 * half;
#pragma unroll
        for (int db = 0; db < DK / 32; ++db)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const float x0 = o[db][4 * q4] * inv, x1 = o[db][4 * q4 + 1] * inv;
            const float x2 = o[db][4 * q4 + 2] * inv, x3 = o[db][4 * q4 + 3] * inv;
            const size_t d = at + 32 * db + 8 * q4;
            if (a.out_f32) {
              *(float4*)((float*)a.out + d) = make_float4(x0, x1, x2, x3);
            } else {
              uint2 pk;
              pk.x = f32_to_bf16_bits(x0) | (f32_to_bf16_bits(x1) << 16);
              pk.y = f32_to_bf16_bits(x2) | (f32_to_bf16_bits(x3) << 16);
              *(uint2*)((bf16_t*)a.out + d) = pk;
            }
          }
      }
    }
  }
}

}  // namespace lisa
