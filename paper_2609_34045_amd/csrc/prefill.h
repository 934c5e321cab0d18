// Internal interface of the chunked-prefill path (matrix cores).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"

namespace kf {

struct PrefillArgs {
  int H, nq, nkv, hd, F;
  float eps;
  int T;          // tokens in the chunk
  int pos0;       // position of the first token
  int user;       // the user's row of the KV cache
  KvPages kv;
  const float* rope_cos;  // [max_ctx][hd/2]
  const float* rope_sin;
  int* err_flag;  // sticky error bits (kErrF16Range for an fp16 activation, key or value out of range)
  hipStream_t stream;
};

struct PrefillLayer {
  const uint16_t *wqkv, *wo, *wg, *wu, *wd, *g_attn, *g_mlp;
  const uint16_t *g_qn, *g_kn;  // per-head q / k norm gains (qk_norm blocks), else NULL
  uint16_t* kc;  // K cache of this layer (fp16 bits), pages as in KvPages
  uint16_t* vc;
  void* out;     // hidden output after this layer (last layer only), else NULL
  int out_bf16;
  // The stage's input (first layer only; exactly one set): hidden rows, fp32 or bf16, or token ids, rows of embed
  const void* src;
  int src_bf16;
  const int32_t* tokens;
  const uint16_t* embed;
  int vocab;
};

// Matrix-core GEMM of the prefill projections (gemm.hip); K must be a multiple
// of 64 (the stage's hidden, ffn and query widths are), else hipErrorInvalidValue.
//   kGemmResidF32   C[M][N] += A W^T (unsplit; the residual stream)
//   kGemmSwiGLU     Cb[M][N/2] = silu(gate) * up in fp16, W the gate rows and W2 the up rows
//   kGemmPartialF32 K slice ks to C + ks*M*N (plain stores); the consumer adds the
//                   plan's slices in order
//   kGemmLogits     C[r][N] = row_scale[r] A W^T; kGemmLogitsSplit: with each row of A in two
//                   parts (launch_head_logits)
enum GemmEpi : int { kGemmResidF32 = 1, kGemmSwiGLU = 2, kGemmPartialF32 = 3, kGemmLogits = 4, kGemmLogitsSplit = 5 };
constexpr int kGemmMaxSlices = 8;  // K slices that the consuming kernels add
// Tile shape and K slices of one product.  `part_elems`: fp32 values that the slices may take.
struct GemmPlan {
  int tile, slices;
};
GemmPlan gemm_plan(int epi, int M, int N, int K, int64_t part_elems);
hipError_t launch_gemm(int epi, const GemmPlan& plan, const uint16_t* A, const uint16_t* W, const uint16_t* W2, int M,
                       int N, int K, float* C, uint16_t* Cb, int* err_flag, hipStream_t s);

// Logits of many rows: logits[rows][N] = RMSNorm(in; gain) W^T on the matrix cores, for
// up to kHeadChunk fp32 rows (2 kHeadChunk bf16 rows when gain is NULL, i.e. folded into W).
// a: [2 kHeadChunk][K] fp16 and row_scale: kHeadScaleBytes are workspace; tile: one of kTiles, or -1 for the plan's.
constexpr int kHeadChunk = 256;  // 8B head: a chunk of 256 fp32 rows takes 550 us, two of 128 rows 600
constexpr int kHeadScaleBytes = 2 * kHeadChunk * (sizeof(double) + sizeof(int));
hipError_t launch_head_logits(const void* in, int in_bf16, const uint16_t* gain, const uint16_t* w, int rows, int N,
                              int K, float eps, uint16_t* a, double* row_scale, float* logits, int* err_flag,
                              hipStream_t s, int tile = -1);

// Device workspace, grown on demand to the largest chunk seen and laid out anew for each chunk.
struct PrefillWorkspace {
  int64_t cap = 0;  // bytes at mem
  bool refused = false;  // the device had not the memory for more
  char* mem = nullptr;
  float* x = nullptr;      // [T][H] residual stream
  uint16_t* xn = nullptr;  // [T][H] normalised, fp16
  float* part = nullptr;   // split-K partial sums [slices][T][N] of the last split projection, or attention partials
  int64_t part_elems = 0;  // values at part
  GemmPlan qkv, oproj, gateup, down;  // the chunk's projections
  int attn_z = 1;                     // key splits of its attention
  int pending = 0;         // slices of the down projection in `part` not yet added to x
  uint16_t* q = nullptr;   // [T][nq][hd] rotated queries, fp16
  uint16_t* o = nullptr;   // [T][nq hd] attention output, fp16
  uint16_t* act = nullptr; // [T][F] SwiGLU output, fp16
};

// Bytes of the no-allocation prefill's scratch array (a 512-token chunk of the 70B shape needs 132 MiB).
constexpr int64_t kPrefillScratchBytes = 144LL << 20;

// Device bytes for a chunk of a.T tokens: what it needs at least, the same for shorter ones
// too, what the plans of all of these would use, and what its own plan would.
struct PrefillSizes {
  int64_t least, shorter, full, own;
};
PrefillSizes prefill_sizes(const PrefillArgs& a);
// Drains the stream (its work may still use the buffer to be replaced) and allocates;
// hipErrorOutOfMemory where the device has not the memory.
hipError_t prefill_grow(void** mem, int64_t bytes, hipStream_t s);
// Grows ws to hold a chunk of a.T tokens, and those of fewer, and lays it out for this one; with
// less room for partial sums, and so fewer slices, where the device has not the memory for all.
hipError_t prefill_reserve(PrefillWorkspace& ws, const PrefillArgs& a,
                           hipError_t (*grow)(void** mem, int64_t bytes, hipStream_t s) = prefill_grow);
void prefill_free(PrefillWorkspace& ws);
// Device bytes a chunk of a.T tokens needs at least; a chunk that needs no more can be laid
// out in `bytes` at `base` (256-byte aligned; ws does not own them).
int64_t prefill_ws_bytes(const PrefillArgs& a);
void prefill_carve(PrefillWorkspace& ws, char* base, int64_t bytes, const PrefillArgs& a);
hipError_t prefill_layer(PrefillWorkspace& ws, const PrefillArgs& a, const PrefillLayer& l, const Tracer& tr);

}  // namespace kf
