// Regression term of the knowledge-distillation loss (Sec. 5.1 "Training strategy"; App. C.1
// "Huber loss function"): for one LiSA layer, the mean over the visible entries of
//   L_delta(a, t) = (a - t)^2 / 2            if |a - t| <= delta
//                   delta (|a - t| - delta / 2) otherwise,
// a = A_n of the student, t = A_n^* of the teacher.  Two passes over nothing but the two score
// tensors: HBM-bound, 2 x 2 bytes per visible entry.
//
// k_kd_huber_tiles (tiled layout) and k_kd_huber_rows (row-major): lanes take pieces of 16 bytes, float32 within a piece,
// float64 from there on; one partial sum per workgroup, in a fixed place.  k_kd_huber_finish: one workgroup adds the partial sums in a fixed
// order (the result does not depend on scheduling) and writes
//   out[0] = (accumulate ? out[0] : 0) + weight * mean,   out[1] = mean
// so that L_KD = (1 / |S|) sum over the layers of S is |S| calls with weight 1 / |S|.
#pragma once
#include "lisa_types.h"

namespace lisa {

constexpr int KD_UN = 2;       // pieces of a lane whose loads are in flight together, tiled scores
constexpr int KD_ROW_UN = 4;   // row-major scores

// 16 bytes of a score tensor, read once by this kernel: a non-temporal load
template <class P>
__device__ __forceinline__ uint4 kd_ld16(const P* p) {
  typedef unsigned kd_u32x4 __attribute__((ext_vector_type(4)));
  const kd_u32x4 v = __builtin_nontemporal_load((const kd_u32x4*)p);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

// How the lanes of k_kd_huber_rows go over the pieces: number q in [0, heads * pairs * pieces) is piece k of the row pair p of
// head bh, k fastest.  A lane goes on by 256 numbers KD_ROW_UN times, then to the next share of its workgroup; the steps are
// given in the same numbering.
struct KdStep {
  int bh, p, k;
};
struct KdWalk {
  int n_heads, n_pairs, pieces;      // B * H, (Lq + 1) / 2, pieces of a pair of rows
  KdStep next, share;
};

// Elements of a line of 128 bytes; (keys + pad) / line lines hold a row's keys wherever the row starts.
template <typename S>
constexpr int kd_line() { return 128 / (int)sizeof(S); }
__host__ __device__ inline unsigned kd_pad(int Lk, int line) { return Lk % line ? 2 * line - 2 : line - 1; }

struct KdArgs {
  const void* a;          // student scores
  const void* t;          // teacher scores, same layout
  double* part;           // [n_blocks] partial sums
  double* out;            // [2]
  int B, H, Lq, Lk, causal, tiled;
  float delta, weight;
  int accumulate, n_blocks;
  long long n_rows;       // B * H * Lq
  KdWalk walk;            // row-major scores
  int parts;              // tiled scores: shares of a pair of row blocks
  double count;           // visible entries of the whole tensor
};

__device__ __forceinline__ float huber1(float a, float t, float delta) {
  const float d = fabsf(a - t), m = fminf(d, delta);       // (m = d: d * d / 2)
  return m * (d - 0.5f * m);
}

// The sum of a workgroup's 256 lanes, in a fixed order (thread 0 has it).
__device__ __forceinline__ double kd_block_sum(double acc) {
  __shared__ double s_part[4];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = acc;
  __syncthreads();
  return (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
}

// Half scores [B, n_rb, n_kt, H, 16, 32]: the visible tiles of a row block (key tiles 0 .. last, all heads)
// are one run of consecutive KB in each tensor.  A workgroup takes a long and a short row block
// at a time (equal work), a wave every fourth KB of the run, KD_UN of them in flight; the
// loads of the run's tail are clamped, not branched around (a load behind a branch makes the
// compiler wait for all earlier ones), and count nothing.  Tiles above the diagonal are not read.
// (few pairs: each is cut into `parts` interleaved shares of its runs, so that the grid has work)
__global__ __launch_bounds__(256) void k_kd_huber_tiles(KdArgs g) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int shift = g.Lk - g.Lq;
  const int n_rb = (g.Lq + 15) / 16, n_kt = (g.Lk + 31) / 32;
  const half_t* a = (const half_t*)g.a;
  const half_t* t = (const half_t*)g.t;
  double acc = 0.0;
  const int n_half = (n_rb + 1) / 2, parts = g.parts;
  const long long n_pairs = (long long)g.B * n_half;
  for (long long item = blockIdx.x; item < n_pairs * parts; item += gridDim.x) {
    const long long pair = item / parts;
    const int part = (int)(item % parts), kw = 4 * parts;   // this wave: every kw-th KB from 4 part + wv
    const int b = (int)(pair / n_half), p = (int)(pair % n_half);
#pragma unroll 1
    for (int side = 0; side < 2; ++side) {
      const int rb = side ? p : n_rb - 1 - p;
      if (side && rb >= n_rb - 1 - p) break;               // (the middle block of an odd count is alone)
      const int i_last = min(16 * rb + 15, g.Lq - 1);
      const int n_keys = g.causal ? min(g.Lk, i_last + 1 + shift) : g.Lk;
      const int run = (n_keys + 31) / 32 * g.H;            // KB of this row block that hold visible entries
      if (run <= 0) continue;
      const size_t base = ((size_t)b * n_rb + rb) * n_kt * g.H * 512 + lane * 8;
      const int i = 16 * rb + (lane >> 2);
      const int vis_row = i < g.Lq ? (g.causal ? min(g.Lk, i + 1 + shift) : g.Lk) : 0;
      for (int k0 = 4 * part + wv; k0 < run; k0 += kw * KD_UN) {
        uint4 av[KD_UN], tv[KD_UN];
#pragma unroll
        for (int u = 0; u < KD_UN; ++u) {
          const size_t at = base + (size_t)min(k0 + kw * u, run - 1) * 512;
          av[u] = kd_ld16(a + at);
          tv[u] = kd_ld16(t + at);
        }
#pragma unroll
        for (int u = 0; u < KD_UN; ++u) {
          const int k = k0 + kw * u;
          const int j8 = 32 * (k / g.H) + 8 * (lane & 3);
          const int nvis = k < run ? vis_row : 0;
          float sm = 0.f;
          const half_t* ah = (const half_t*)&av[u];
          const half_t* th = (const half_t*)&tv[u];
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (j8 + e < nvis) sm += huber1((float)ah[e], (float)th[e], g.delta);
          acc += (double)sm;
        }
      }
    }
  }
  acc = kd_block_sum(acc);
  if (threadIdx.x == 0) g.part[blockIdx.x] = acc;
}

// Row-major scores of element type S (half_t or float), rows of any length.  The tensors are read as pieces of 16 bytes at
// 16-byte boundaries whatever Lk is: both have the same layout, so a piece of one belongs to the same elements as that of
// the other, and what of a piece lies outside its row's visible keys is not summed.  A row's pieces are those of the lines
// of 128 bytes that hold its keys, so that the 64 pieces of a wave are always 8 whole lines (numbered from the row's first
// piece a wave's loads took parts of 9 lines: LLaMA2-7B heads, 2 x 2112 tokens, 102 against 96 us).  Row p and row
// Lq - 1 - p together have about as many for every p: numbering (head, pair, piece) deals equal work to all lanes without
// a division per piece.  HBM-bound.  Against a wave per row, which took rows with Lk % 8 != 0 element by element:
// LLaMA3-8B heads, 2 x 1611 tokens, 202 -> 60 us (5.5 TB/s), LLaMA2-7B, 2 x 2112 (whole pieces before) 97 -> 96 us (5.9).
template <typename S>
__global__ __launch_bounds__(256) void k_kd_huber_rows(KdArgs g) {
  constexpr int E = 16 / sizeof(S), G = kd_line<S>();       // elements of a piece, of a line
  const S* a = (const S*)g.a;
  const S* t = (const S*)g.t;
  const KdWalk w = g.walk;
  const int shift = g.Lk - g.Lq;
  const unsigned long long n_elems = (unsigned long long)g.n_rows * (unsigned)g.Lk;
  const unsigned long long last = n_elems / E - 1;          // the last whole piece (n_elems >= E)
  const unsigned pad = kd_pad(g.Lk, G);
  const unsigned first = blockIdx.x * (256 * KD_ROW_UN) + threadIdx.x;
  int k = (int)(first % w.pieces), bh, p;
  {
    const unsigned rest = first / w.pieces;
    p = (int)(rest % w.n_pairs);
    bh = (int)(rest / w.n_pairs);
  }
  double acc = 0.0;
  while (bh < w.n_heads && n_elems >= E) {
    uint4 av[KD_ROW_UN], tv[KD_ROW_UN];
    unsigned rel[KD_ROW_UN], len[KD_ROW_UN];                        // element e counts where rel + e < len
#pragma unroll
    for (int u = 0; u < KD_ROW_UN; ++u) {
      const int p1 = g.Lq - 1 - p;
      const unsigned n0 = g.causal ? p + 1 + shift : g.Lk, n1 = p1 > p ? (g.causal ? p1 + 1 + shift : g.Lk) : 0;
      const unsigned c0 = (n0 + pad) / G * (G / E);
      const bool second = (unsigned)k >= c0;
      const unsigned piece = second ? k - c0 : k;           // of its row
      const unsigned long long start = ((unsigned long long)(unsigned)bh * (unsigned)g.Lq + (second ? p1 : p)) * (unsigned)g.Lk;
      const unsigned n = second ? n1 : n0;
      const unsigned long long at = start / G * (G / E) + piece, end = (start + n - 1) / E;
      rel[u] = piece * E - (unsigned)start % G;             // (below 0: elements of the row before)
      len[u] = bh < w.n_heads && at <= last ? n : 0;
      const size_t from = min(min(at, end), last) * E;      // (nothing behind the row's last piece is fetched)
      av[u] = kd_ld16(a + from);
      tv[u] = kd_ld16(t + from);
      const KdStep st = u + 1 < KD_ROW_UN ? w.next : w.share;
      k += st.k;
      p += st.p;
      bh += st.bh;
      if (k >= w.pieces) { k -= w.pieces; ++p; }
      if (p >= w.n_pairs) { p -= w.n_pairs; ++bh; }
    }
#pragma unroll
    for (int u = 0; u < KD_ROW_UN; ++u) {
      const S* ae = (const S*)&av[u];
      const S* te = (const S*)&tv[u];
      float sm = 0.f;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const float h = huber1((float)ae[e], (float)te[e], g.delta);
        sm += rel[u] + e < len[u] ? h : 0.f;
      }
      acc += (double)sm;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < n_elems % E) {       // elements behind the last whole piece
    const unsigned long long x = n_elems / E * E + threadIdx.x;
    const int i = (int)(x / g.Lk % g.Lq), j = (int)(x % g.Lk);
    if (!g.causal || j <= i + shift) acc += (double)huber1(elem<S>::load(a + x), elem<S>::load(t + x), g.delta);
  }
  acc = kd_block_sum(acc);
  if (threadIdx.x == 0) g.part[blockIdx.x] = acc;
}

__global__ __launch_bounds__(256) void k_kd_huber_finish(KdArgs g) {
  double s = 0.0;
  for (int k = threadIdx.x; k < g.n_blocks; k += 256) s += g.part[k];
  s = kd_block_sum(s);
  if (threadIdx.x == 0) {
    const double mean = s / g.count;
    g.out[0] = (g.accumulate ? g.out[0] : 0.0) + (double)g.weight * mean;
    g.out[1] = mean;
  }
}

}  // namespace lisa
