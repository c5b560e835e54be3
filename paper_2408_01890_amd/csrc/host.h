// Host-side helpers shared by the translation units of the library: status reporting, stage timing and
// the launchers that live in files of their own (their kernels have many instantiations, which
// compile side by side that way).
#pragma once
#include "../../include/lisa.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>

#include "kernels_decode.h"
#include "kernels_prefill.h"
#include "kernels_scores_mfma.h"

namespace lisa {

constexpr int kComputeUnits = 256;   // MI355X

inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline float pick_scale(float given, int n) { return given > 0.f ? given : 1.0f / std::sqrt((float)n); }

// Prefill scores that the bf16 and half matrix-core kernels can read and write: 8 at a time, at 16-byte boundaries
// (whole tiles always are).
inline bool score_rows_aligned(const lisa_desc* d) { return d->score_tiled ? d->Lk >= 8 : d->Lk % 8 == 0; }

int hip_fail(hipError_t e);          // remembers the error's text for lisa_last_hip_error()
int check_launch();

// ---- optional stage timing (lisa_profile_*) -------------------------------------------
struct ProfRec {
  const char* name;
  hipEvent_t beg, end;
};
// Brackets the launches made while it is alive with two events on their stream.
struct StageScope {
  hipStream_t st;
  ProfRec rec{nullptr, nullptr, nullptr};
  StageScope(const char* name, hipStream_t s);
  ~StageScope();
};

// launch_prefill.hip, launch_decode.hip, launch_scores.hip
template <int NG, int HPW, int NW>
int launch_prefill_fused_fs(const lisa_desc* d, const PrefillArgs& a, int slices, hipStream_t st);
int launch_decode_part(const lisa_desc* d, bool lisa_layer, DecodeArgs a, hipStream_t st);
// launch_stack.hip
bool stack_chained_ok(const lisa_desc* d);
size_t stack_chained_bytes(const lisa_desc* d);
// Scratch of a single layer on the kernels of the stacks at most: with what synth_relu_ffn() adds behind it
// (under 64 KB here) it fits the buffer of lisa_attn_decode_static.
constexpr size_t kDecodeSpreadMaxBytes = LISA_STATIC_SCRATCH_BYTES - 128 * 1024;
bool decode_spread_fits(const lisa_desc* d);
bool decode_spread_ok(const lisa_desc* d, bool lisa_layer);
size_t decode_spread_bytes(const lisa_desc* d);
FfnOperands decode_spread_operands(const lisa_desc* d, const bf16_t* w1, const bf16_t* w2, void* workspace);
int run_decode_spread(const lisa_desc* d, bool lisa_layer, const DecodeArgs& da, void* out, void* workspace,
                      hipStream_t st);
int run_stack_chained(const lisa_desc* d, const lisa_stack_layer* layers, int n_layers, void* const rows[2],
                      void* workspace, hipStream_t st);
// launch_f32.hip
bool f32_attn_ok(const lisa_desc* d);
int run_f32_attn(const lisa_desc* d, const void* q, const void* k, const void* v, const float* given, int row0, int n_rows,
                 void* scores, void* out, hipStream_t st);
int f32_attn_order(const lisa_desc* d, int n_rows, int parts);
int f32_chunk_rows(const lisa_desc* d);
size_t f32_chunk_bytes(const lisa_desc* d);
bool f32_scores_ok(const lisa_desc* d);
int run_f32_scores(const lisa_desc* d, const void* q_lr, const void* k_lr, const void* prev, const void* w1,
                   const void* w2, void* scores, float* exact, int row0, int n_rows, hipStream_t st);
// launch_split.hip
bool bf16_ragged_rows(const lisa_desc* d);
bool split_attn_ok(const lisa_desc* d);
bool split_scores_ok(const lisa_desc* d);
int split_chunk_rows(const lisa_desc* d);
size_t split_bytes(const lisa_desc* d);
int run_split_prepare(const lisa_desc* d, const void* q_lr, const void* k_lr, const void* w1, const void* w2, void* workspace,
                      hipStream_t st);
int run_split_scores(const lisa_desc* d, const void* prev, void* scores, void* workspace, int row0, int n_rows, hipStream_t st);
int run_split_attn(const lisa_desc* d, const void* q, const void* k, const void* v, const float* given, bool given_tiled,
                   int row0, int n_rows, void* scores, void* out, hipStream_t st);
int split_attn_order(const lisa_desc* d, int n_rows, int parts);
FfnImage scores_mfma_image(const lisa_desc* d, const void* w1, const void* w2);
int launch_scores_mfma_kernel(const lisa_desc* d, const ScoresMfmaArgs& a, hipStream_t st);

}  // namespace lisa
