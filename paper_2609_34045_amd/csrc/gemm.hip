// Prefill projections on the matrix cores: C[M][N] (+)= A[M][K] x W[N][K]^T.
//
// A is fp16 activations, W is fp16 weights (converted from the model's bf16
// once, when the stage is created), both K-contiguous; the product runs on v_mfma_f32_32x32x16_f16 with
// fp32 accumulation.  At a 512-token chunk the projections are large enough
// to be bound by the matrix cores, which sets the tile shape:
//   * 256 x 256 x 64 workgroup tiles, eight waves (two per SIMD) of 128 x 64,
//     8 accumulator blocks each: per K step a wave reads 24 KB of fragments
//     from LDS for 32 MFMAs.  Two waves per SIMD let one issue MFMAs while the
//     other waits on LDS or the barrier (four waves of 128 x 128 measured 4-5%
//     slower);
//   * narrower tiles (224, 160 or 128 columns) where they fill whole rounds of
//     the 256 CUs in less time (the 70B gate/up shape: 512 tiles of 224 columns
//     in 2 rounds, against 448 of 256 whose second round is three quarters
//     full): eight waves, the wide and the narrow ones one of each per SIMD;
//   * up to 128 rows, where the stream of the weights bounds the product, tiles
//     of 32, 64 or 128 rows in a kernel of their own (gemm_rows_kernel);
//   * operands go from global memory straight into LDS rings with
//     global_load_lds (no register staging).  A 64-deep K step makes each load
//     instruction fetch 8 rows x 128 B, i.e. whole cache lines; 32-deep steps
//     fetched 16 half lines per instruction and ran the 70B gate/up shape
//     5-7% slower.  The weights, which stream from HBM, get a 3-stage ring
//     (loads run two K steps ahead), the activations, which stay in L2, a
//     2-stage one: 160 KB together, 2% faster on that shape than 2 stages of
//     both (the whole 70B chunk 1%, the Qwen3-32B-shaped one 2.5%);
//   * chunks are XOR-swizzled within a row so that fragment reads are free of
//     bank conflicts;
//   * each wave reads the fragments of the next 16-wide K slice while the
//     MFMAs of the current one run;
//   * a product without enough tiles is split along K over several workgroups
//     so that the grid covers the 256 CUs; the slices are stored whole for the
//     consuming kernel to add in order (kGemmPartialF32).  gemm_plan chooses
//     the tile and the slices.
// Operand fragment layout of v_mfma_f32_32x32x16_f16 (lane l of 64):
//   A: row l%32, k = 8*(l/32) .. +7      B: column l%32, k = 8*(l/32) .. +7
//   D: element v (0..15) at row 8*(v/4) + 4*(l/32) + v%4, column l%32
#include "kernels.h"
#include "prefill.h"

namespace kf {
namespace {

typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr;

constexpr int BK = 64;             // K step
constexpr int ROW_BYTES = BK * 2;  // bytes per tile row and step: a cache line
constexpr int CH = BK / 8;         // 16-byte chunks per tile row
constexpr int SS = BK / 16;        // 16-wide K slices (MFMA steps) per K step

__device__ __forceinline__ f32x16 mfma32(v4u a, v4u b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}

// Chunk c of tile row r is stored at slot c ^ f(r) of that row, f(r) = r % 8 ^
// (r/8) % 2: any 8 consecutive rows hit distinct 16-byte bank groups of a
// 32-bank LDS, and any 16 consecutive rows of a 64-bank one, so the fragment
// reads (one row per lane) are free of bank conflicts.
__device__ __forceinline__ int swz(int r, int c) { return c ^ ((r & 7) ^ ((r >> 3) & 1)); }

// Wait until at most N vector-memory operations of this wave are outstanding.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | (0x7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}

// Wait until this wave's LDS reads have returned (global loads may stay in flight).
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(0xF | (0x7 << 4) | (0x3 << 14)); }

// Workgroup barrier that orders LDS accesses without waiting on outstanding
// global loads (the compiler may not move memory operations across it).
__device__ __forceinline__ void block_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

struct Params {
  const uint16_t* A;
  const uint16_t* W;
  const uint16_t* W2;
  int M, N, K;
  int splitk;  // K slices (1: read-modify-write or SwiGLU epilogue)
  float* C;
  uint16_t* Cb;
  int* err_flag;
  // logits only:
  int rows_out;             // rows of the output (M counts the rows of A)
  const double* row_scale;  // factor of each output row; its sign is set for the rows of wide_rows
  int kstride;              // K steps are taken in the order 0, kstride, 2 kstride, .. (mod their number)
  int fold;                 // K steps that an accumulator runs over (Accum)
  const void* in;           // the rows themselves, fp32 or (in_bf16) bf16, the gain that is not folded into W,
  int in_bf16;              // and the exponent that scales each row (head_rows_kernel)
  const uint16_t* gain;
  const int* row_exp;
};

// Rows of A per output row: the logits of fp32 rows take each row as two fp16
// parts, in 32-row blocks of high parts, each followed by the block of the low
// parts, that add into one accumulator.
constexpr int parts_of(int epi) { return epi == kGemmLogitsSplit ? 2 : 1; }
constexpr bool is_logits(int epi) { return epi == kGemmLogits || epi == kGemmLogitsSplit; }

// Accumulators of a wave's MB x JW output blocks.
template <int EPI, int MB, int JW>
struct Accum {
  f32x16 acc[MB][JW] = {};
  __device__ __forceinline__ void begin_step(const Params&) {}
};

// Those of the logits.  A matrix instruction rounds into its accumulator twice, so
// one chain of them over all of K loses what the fp32 tree sums of a GEMV keep: against
// 64-bit sums over the stored matrix, K = 4096, fp32 rows 5.8e-7 (GEMV 1.2e-7),
// bf16 rows 4.2e-7 (1.0e-7).  An accumulator therefore runs over p.fold steps and is
// then added into `sum`, keeping what that sum rounded off.
template <int MB, int JW>
struct LogitAccum {
  f32x16 acc[MB][JW] = {}, sum[MB][JW] = {};
  int left = 0;  // steps until the next fold
  __device__ __forceinline__ void begin_step(const Params& p) {
    if (left-- > 0) return;
    left = p.fold - 1;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < JW; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float s = sum[i][j][v], a = acc[i][j][v], t = s + a;
          acc[i][j][v] = a - (t - s);  // (no infinities here: wide_rows takes their rows)
          sum[i][j][v] = t;
        }
  }
};
template <int MB, int JW>
struct Accum<kGemmLogits, MB, JW> : LogitAccum<MB, JW> {};
template <int MB, int JW>
struct Accum<kGemmLogitsSplit, MB, JW> : LogitAccum<MB, JW> {};

// Large tiles: TM rows (256 or 128) x 32 NB columns, eight waves (two per SIMD).
// LDS ring depths: activation loads run up to ring_a K steps ahead, weight
// loads up to ring_w; as deep as 160 KB allow (with the depths of the widest, 2
// and 3, tiles of 128 columns waited on their activations: 8B-shaped gate/up
// at 200 rows 77.0 -> 69.2 us).
constexpr int NW = 8;
constexpr int ring_a(int TM, int NB) { return TM == 256 && NB >= 7 ? 2 : 3; }
constexpr int ring_w(int NB) { return NB == 4 ? 4 : 3; }
constexpr int a_stage(int TM) { return TM * ROW_BYTES; }
constexpr int w_stage(int NB) { return 32 * NB * ROW_BYTES; }

// Logits of the rows that their fp16 parts do not hold (head_rows_kernel), in fp32, by
// the launch's workgroups past its tiles: wave `wave` of `waves`.  Such rows are the
// exception: where there are none these workgroups end at once, beside the tiles' (a launch of
// their own cost 3 to 5 us).  Otherwise they are bound by the stream of the matrix, four rows a
// pass (8B head: 220 to 270 us).  A wave takes four columns at a time, so that the rows' values, which come from the
// caches, serve four of the matrix's; eight products are added pairwise, and a lane adds
// K / 512 of these.
constexpr int kWideCols = 4, kWideWorkgroups = 256;
__device__ __forceinline__ void wide_rows(const Params& p, int lane, int wave, int waves) {
  constexpr int R = 4, C = kWideCols;
  const int H = p.K, last = p.N;
  bool nan = false;
  for (int b = 0; b < p.rows_out; b += 64) {
    uint64_t todo = __ballot(b + lane < p.rows_out && __builtin_signbit(p.row_scale[min(b + lane, p.rows_out - 1)]));
    while (todo) {
      int r[R], e[R];
      const uint2* row[R];
      int n = 0;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        r[i] = i && !todo ? r[i > 0 ? i - 1 : 0] : b + __builtin_ctzll(todo);
        if (todo) ++n;
        todo &= todo - (todo != 0);
        e[i] = p.row_exp[r[i]];
        row[i] = reinterpret_cast<const uint2*>(p.in) + (int64_t)r[i] * (p.in_bf16 ? H / 4 : H / 2);
      }
      for (int c0 = C * wave; c0 < last; c0 += C * waves) {
        float sum[C][R] = {};
        for (int k = lane; k < H / 8; k += 64) {
          // every load before a use: a branch on the rows' type would wait for each row in turn
          h8 wk[C];
#pragma unroll
          for (int c = 0; c < C; ++c) wk[c] = reinterpret_cast<const h8*>(p.W + (int64_t)min(c0 + c, last - 1) * H)[k];
          uint2 raw[R][4];  // 8 values: 4 words of bf16 (twice), or 8 of fp32
#pragma unroll
          for (int i = 0; i < R; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) raw[i][j] = row[i][p.in_bf16 ? 2 * k + (j & 1) : 4 * k + j];
          float g[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) g[j] = p.gain ? __uint_as_float((uint32_t)p.gain[8 * k + j] << 16) : 1.f;
#pragma unroll
          for (int i = 0; i < R; ++i) {
            float x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const uint32_t half = j & 2 ? raw[i][j / 4].y : raw[i][j / 4].x, word = j & 1 ? raw[i][j / 2].y : raw[i][j / 2].x;
              x[j] = ldexpf(__uint_as_float(p.in_bf16 ? (j & 1 ? half & 0xffff0000u : half << 16) : word) * g[j], e[i]);
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
              float q[4];
#pragma unroll
              for (int j = 0; j < 4; ++j) q[j] = fmaf((float)wk[c][2 * j], x[2 * j], (float)wk[c][2 * j + 1] * x[2 * j + 1]);
              sum[c][i] += (q[0] + q[1]) + (q[2] + q[3]);
            }
          }
        }
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int i = 0; i < R; ++i) {
            float t = sum[c][i];
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) t += __shfl_xor(t, o);
            if (lane == 0 && i < n && c0 + c < last) {
              const float y = (float)((double)t * fabs(p.row_scale[r[i]]));
              nan |= y != y;
              p.C[(int64_t)r[i] * p.N + c0 + c] = y;
            }
          }
      }
    }
  }
  raise_err(p.err_flag, nan, kErrNaNLogit);
}

// Epilogue of one wave's accumulators: MB 32-row blocks from output row row0
// times JW 32-column blocks from block bw0 of the tile at column n0.  Lane l
// holds column l % 32 of each block.
template <int EPI, int MB, int JW>
__device__ __forceinline__ void store_tile(const Params& p, const Accum<EPI, MB, JW>& sums, int lane, int row0, int n0,
                                           int bw0, int ks) {
  const auto& acc = sums.acc;
  const int rl = lane & 31, rq = 4 * (lane >> 5);
  if (EPI == kGemmSwiGLU) {
    // Each 32-column block holds 16 outputs: columns 0-15 their gate rows,
    // 16-31 their up rows.  Lanes c and c ^ 16 exchange values; the gate lane
    // writes elements v = 0..7 of the pair, the up lane v = 8..15.
    bool bad = false;
    const bool gl = (lane & 16) == 0;
    const int nout = p.N >> 1;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < JW; ++j) {
        float pr[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) pr[v] = __shfl_xor(acc[i][j][v], 16);
        const int col = (n0 >> 1) + 16 * (bw0 + j) + (lane & 15);
#pragma unroll
        for (int v = 0; v < 8; ++v) {
          const int vv = gl ? v : v + 8;
          const float g = gl ? acc[i][j][v] : pr[v + 8], u = gl ? pr[v] : acc[i][j][v + 8];
          const int row = row0 + 32 * i + 8 * (vv >> 2) + rq + (vv & 3);
          if (row < p.M && col < nout) p.Cb[(int64_t)row * nout + col] = f16_checked(g / (1.0f + expf(-g)) * u, bad);
        }
      }
    raise_err(p.err_flag, bad, kErrF16Range);
  } else if constexpr (is_logits(EPI)) {
    bool nan = false;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      // every factor before the first is used (the tile's rows past the output lie in the array too)
      double scale[16];
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        const double2 two = *reinterpret_cast<const double2*>(p.row_scale + row0 + 32 * i + 8 * (v >> 2) + rq + (v & 3));
        scale[v] = two.x;
        scale[v + 1] = two.y;
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        if (row0 + 32 * i + 8 * (v >> 2) >= p.rows_out) break;
        const int row = row0 + 32 * i + 8 * (v >> 2) + rq + (v & 3);
        const bool skip = __builtin_signbit(scale[v]);
#pragma unroll
        for (int j = 0; j < JW; ++j) {
          const int col = n0 + 32 * (bw0 + j) + rl;
          const float y = (float)(((double)sums.sum[i][j][v] + (double)acc[i][j][v]) * scale[v]);
          if (row < p.rows_out && col < p.N && !skip) {
            nan |= y != y;
            p.C[(int64_t)row * p.N + col] = y;
          }
        }
      }
    }
    raise_err(p.err_flag, nan, kErrNaNLogit);
  } else {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = row0 + 32 * i + 8 * (v >> 2) + rq + (v & 3);
        if (row >= p.M) continue;
#pragma unroll
        for (int j = 0; j < JW; ++j) {
          const int col = n0 + 32 * (bw0 + j) + rl;
          if (col >= p.N) continue;
          float* c = p.C + (int64_t)row * p.N + col;
          if (EPI == kGemmResidF32) *c += acc[i][j][v];
          else c[(int64_t)ks * p.M * p.N] = acc[i][j][v];
        }
      }
  }
}

// One wave's share of a tile: the K loop and the epilogue for MB 32-row A
// blocks from tile row am0 times JW 32-column W blocks from block bw0.  Every
// wave also issues its share of the tile loads: TM / 64 of the A tile and LW of
// the W tile per stage.
template <int EPI, int TM, int NB, int MB, int JW, int LW>
__device__ __forceinline__ void gemm_wave(const Params& p, uint8_t* smem, const uint16_t* const (&asrc)[TM / 64],
                                          const uint16_t* const (&wsrc)[4], int nk, int wave, int lane,
                                          int m0, int n0, int am0, int bw0, int ks) {
  constexpr int SA = ring_a(TM, NB), SW = ring_w(NB);
  constexpr int PA = parts_of(EPI);  // A blocks per accumulator block
  static_assert(MB % PA == 0, "whole output blocks");
  constexpr int SLOTS = MB * JW;  // MFMAs per 16-wide K slice
  constexpr int RD = MB + JW;     // fragment reads per slice
  constexpr int LA = TM / 64;     // A loads per stage
  constexpr int NL = LA + LW;     // direct loads per slice that carries them
  static_assert(RD <= SLOTS && LW <= 4, "a slice's slots issue its reads");

  // Step kt's stages and source; past the last step a load fetches step nk-1 (logits:
  // an earlier step) again, into the stage of the step it stands in for, which is never read.
  auto abuf = [&](int kt) { return smem + (kt % SA) * a_stage(TM); };
  auto wbuf = [&](int kt) { return smem + SA * a_stage(TM) + (kt % SW) * w_stage(NB); };
  auto src_step = [&](int kt) {
    if (is_logits(EPI)) return (int64_t)((unsigned)(kt * p.kstride) % (unsigned)nk) * BK;
    return (int64_t)(kt < nk ? kt : nk - 1) * BK;
  };
  // (named operands: the host pass drops the kernel's launch stub when the
  // builtin's pointer argument is a call expression)
  auto load_one = [&](bool w, int j, int kt) {
    const uint16_t* src = (w ? wsrc[j] : asrc[j]) + src_step(kt);
    uint8_t* dst = (w ? wbuf(kt) : abuf(kt)) + 1024 * (NW * j + wave);
    __builtin_amdgcn_global_load_lds(src, (lds_ptr)dst, 16, 0, 0);
  };

  Accum<EPI, MB / PA, JW> sums;
  auto& acc = sums.acc;

  // The K loop is scheduled by hand: each slice is SLOTS MFMA slots; the
  // first slots also issue the fragment reads for the next slice (and, in the
  // slice after the barrier, the direct loads, spread over the slots).
  const int rl = lane & 31, kh = lane >> 5;
  // fragment read q (0..RD-1) of slice s (16 values of K) of step k: weight
  // block q for q < JW, then A block q-JW
  auto read_frag = [&](int k, int s, int q, v4u (&fa)[MB], v4u (&fw)[JW]) {
    const bool w = q < JW;
    const uint8_t* buf = w ? wbuf(k) : abuf(k);
    const int r = w ? 32 * (bw0 + q) + rl : am0 + 32 * (q - JW) + rl;
    const v4u v = *reinterpret_cast<const v4u*>(buf + r * ROW_BYTES + swz(r, 2 * s + kh) * 16);
    if (w) fw[q] = v;
    else fa[q - JW] = v;
  };
  // One slice: the SLOTS MFMAs on (fa, fw), the reads of the next fragments
  // (slice rs of step rk) into (na, nw), one per slot from slot 0, and
  // optionally the loads of steps ka (A, issued first) and kw (W).
  auto half = [&](const v4u (&fa)[MB], const v4u (&fw)[JW], int rk, int rs, v4u (&na)[MB], v4u (&nw)[JW],
                  bool load, int ka, int kw) {
#pragma unroll
    for (int q = 0; q < SLOTS; ++q) {
      acc[q / JW / PA][q % JW] = mfma32(fa[q / JW], fw[q % JW], acc[q / JW / PA][q % JW]);
      if (q < RD) read_frag(rk, rs, q, na, nw);
      if (load) {
#pragma unroll
        for (int l = q * NL / SLOTS; l < (q + 1) * NL / SLOTS; ++l) load_one(l >= LA, l >= LA ? l - LA : l, l >= LA ? kw : ka);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // Rings: step k's activations live in A stage k % SA, its weights in W
  // stage k % SW.  The fragments of slice s+1 are read while the MFMAs of
  // slice s run.  The barrier before the last slice of step k releases step
  // k+1's data to every wave and hands both of step k's stages (whose last
  // reads were issued in the slice before) to the loads of step k + SA (A) and
  // k + SW (W), which are issued A first.  Past the last step those loads
  // repeat step nk-1 into stages that are not read again, which keeps the loop
  // free of branches and the wait counts fixed.
#pragma unroll
  for (int s = 0; s < SW; ++s) {
    if (s < SA) {
#pragma unroll
      for (int j = 0; j < LA; ++j) load_one(false, j, s);
    }
#pragma unroll
    for (int j = 0; j < LW; ++j) load_one(true, j, s);
  }
  wait_vm<(SA - 1) * LA + (SW - 1) * LW>();  // step 0 has landed
  block_barrier();
  v4u fa[2][MB], fw[2][JW];
#pragma unroll
  for (int q = 0; q < RD; ++q) read_frag(0, 0, q, fa[0], fw[0]);
  static_assert(SS % 2 == 0, "a step starts with its fragments in buffer 0");
  for (int k = 0; k + 1 < nk; ++k) {
    sums.begin_step(p);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s + 1 < SS; ++s)
      half(fa[s & 1], fw[s & 1], k, s + 1, fa[(s + 1) & 1], fw[(s + 1) & 1], false, 0, 0);
    // This wave's loads for step k+1 are complete once only later steps' remain
    // in flight: the A loads of steps k+2 .. k+SA-1 and the W loads of steps
    // k+2 .. k+SW-1, which are the most recent ones (A before W within a step).
    wait_vm<(SA - 2) * (LA + LW) + (SW - SA) * LW>();
    wait_lds();  // this wave's reads of step k's stages have returned (issued a slice ago)
    // Every wave's loads for step k+1 have landed and every wave's reads of
    // step k's stages have returned.  A bare barrier: a fence here would also
    // drain the loads in flight.
    block_barrier();
    half(fa[1], fw[1], k + 1, 0, fa[0], fw[0], true, k + SA, k + SW);
  }
  {
    const int k = nk - 1;
    sums.begin_step(p);
#pragma unroll
    for (int s = 0; s + 1 < SS; ++s)
      half(fa[s & 1], fw[s & 1], k, s + 1, fa[(s + 1) & 1], fw[(s + 1) & 1], false, 0, 0);
#pragma unroll
    for (int q = 0; q < SLOTS; ++q)
      acc[q / JW / PA][q % JW] = mfma32(fa[1][q / JW], fw[1][q % JW], acc[q / JW / PA][q % JW]);
  }
  wait_vm<0>();  // no load may still be writing LDS when the workgroup ends

  store_tile<EPI, MB / PA, JW>(p, sums, lane, (m0 + am0) / PA, n0, bw0, ks);
}

// Tiles of TM rows x 32 NB columns (narrower or lower ones where they fill the
// chip in less time: see gemm_plan).  At 256 rows: with NB = 8 the eight waves
// are 2 x 4 of 128 x 64; with NB = 7 (5) they are 4 x 2 of 64 x 128 (96) and 64
// x 96 (64), so that with waves dealt to the SIMDs round-robin each SIMD holds
// one of each; with NB = 4, 4 x 2 of 64 x 64.  The 128-row tile (2 x 4 waves of
// 64 x 64) serves chunks that end in less than half a 256-row tile (300 rows:
// 70B-shaped gate/up 431 -> 402 us, 32B-shaped down 133 -> 118).
template <int EPI, int TM, int NB>
__global__ __launch_bounds__(64 * NW) void gemm_tile_kernel(const Params p) {
  static_assert(TM == 256 ? NB == 8 || NB == 7 || NB == 5 || NB == 4 : TM == 128 && NB == 8, "tiles");
  constexpr int SA = ring_a(TM, NB), SW = ring_w(NB), LDS = SA * a_stage(TM) + SW * w_stage(NB);
  static_assert(SA >= 2 && SW >= SA && SW <= SA + 1 && LDS <= 160 * 1024, "ring depths");
  // SA A stages, then SW W stages, of rows of CH swizzled 16-byte chunks; both fp16.
  __shared__ __attribute__((aligned(1024))) uint8_t smem[LDS];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int TN = 32 * NB;  // tile columns
  const int mt = (p.M + TM - 1) / TM, nt = (p.N + TN - 1) / TN, ntiles = mt * nt;
  const int nwg = ntiles * p.splitk;
  if constexpr (is_logits(EPI)) {
    if ((int)blockIdx.x >= nwg) return wide_rows(p, lane, NW * (blockIdx.x - nwg) + wave, NW * (gridDim.x - nwg));
  }
  // Tiles sharing a weight panel (same column tile) go to the same XCD, where
  // they reuse it through that XCD's L2 (workgroups are dealt round-robin).
  int bid = blockIdx.x;
  {
    const int x = bid % 8, q = nwg / 8, r = nwg % 8;  // XCD x holds q workgroups, one more while x < r
    bid = x * q + (x < r ? x : r) + bid / 8;
  }
  const int ks = bid % p.splitk, t = bid / p.splitk;
  const int tm = t % mt, tn = t / mt;
  const int m0 = tm * TM, n0 = tn * TN;
  const int K = p.K;
  const int nk_all = K / BK;
  const int k_begin = (int)((int64_t)nk_all * ks / p.splitk), k_end = (int)((int64_t)nk_all * (ks + 1) / p.splitk);
  const int nk = k_end - k_begin;

  // Direct global -> LDS loads: load j of this wave fills the 1 KB of tile rows
  // 8 (NW j + wave) .. + 7; lane l writes row 8 (NW j + wave) + l / 8, slot l % 8,
  // so it fetches the chunk that belongs in that slot (the 8 lanes of a row
  // cover 128 contiguous bytes).
  const int w_rows = EPI == kGemmSwiGLU ? (p.N >> 1) : p.N;
  const uint16_t* asrc[TM / 64];
  const uint16_t* wsrc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = 8 * (NW * j + wave) + lane / CH;
    const int c = swz(r, lane % CH);
    if (j < TM / 64) {
      const int ar = m0 + r < p.M ? m0 + r : p.M - 1;  // rows past M load a valid row; they are never stored
      asrc[j] = p.A + (int64_t)ar * K + (int64_t)k_begin * BK + c * 8;
    }
    // weight tile row r (of the loads a wave issues: below TN); for SwiGLU, each
    // 32-row block holds the gate rows (first 16) and the up rows (last 16) of 16 outputs
    int wr;
    const uint16_t* wb;
    if (EPI == kGemmSwiGLU) {
      wr = (n0 >> 1) + 16 * (r >> 5) + (r & 15);
      wb = (r & 16) ? p.W2 : p.W;
    } else {
      wr = n0 + r;
      wb = p.W;
    }
    if (wr >= w_rows) wr = w_rows - 1;  // columns past N load a valid row; they are never stored
    wsrc[j] = wb + (int64_t)wr * K + (int64_t)k_begin * BK + c * 8;
  }
  // W tile load j of wave w fills rows 8 (8 j + w) ..: each wave issues those below TN
  // (NB = 7: load 3 of waves 0..3; NB = 5: load 2 of waves 0..3).
  if constexpr (TM == 128) {
    gemm_wave<EPI, TM, NB, 2, 2, 4>(p, smem, asrc, wsrc, nk, wave, lane, m0, n0, 64 * (wave / 4), 2 * (wave % 4), ks);
  } else if constexpr (NB == 8) {
    gemm_wave<EPI, TM, NB, 4, 2, 4>(p, smem, asrc, wsrc, nk, wave, lane, m0, n0, 128 * (wave / 4), 2 * (wave % 4), ks);
  } else if constexpr (NB == 4) {
    gemm_wave<EPI, TM, NB, 2, 2, 2>(p, smem, asrc, wsrc, nk, wave, lane, m0, n0, 64 * (wave & 3), 2 * (wave >> 2), ks);
  } else {
    constexpr int J0 = (NB + 1) / 2, J1 = NB / 2;  // blocks of waves 0..3 and 4..7, which also issue as many loads
    if (wave < 4) gemm_wave<EPI, TM, NB, 2, J0, J0>(p, smem, asrc, wsrc, nk, wave, lane, m0, n0, 64 * wave, 0, ks);
    else gemm_wave<EPI, TM, NB, 2, J1, J1>(p, smem, asrc, wsrc, nk, wave, lane, m0, n0, 64 * (wave - 4), J0, ks);
  }
}

// ------------------------------------------------------------------ few rows
// Products over up to 128 rows: bound by the stream of the weights from HBM,
// not by the matrix cores, so the tile is only as tall as the rows (32, 64 or
// 128) and the launch is cut along N and K until every CU streams.  A
// workgroup of WM x WN waves, each with MBW x JW blocks of 32 x 32, takes
// 32 MBW WM rows x 32 JW WN columns of one K slice; both operands go straight
// into one LDS ring of D stages of 64-deep K steps (loads run D - 1 steps
// ahead).  Up to 64 rows the ring leaves room for two workgroups on a CU, so
// one computes while the other waits; at 128 rows, where each weight fragment
// meets four times the products, eight waves share the tile instead.
// Against 256-row tiles (weights cold in HBM, 8B shape): 32 rows, gate/up
// 87 -> 39 us (6.0 TB/s), QKV 34.5 -> 11, output 32 -> 8.4, down 40 -> 20; 64
// rows 89 -> 42, 34 -> 12, 33 -> 9.6, 41 -> 22; 128 rows 90 -> 50, 34 -> 16,
// 33 -> 14, 43 -> 31.  Tried and no faster: deeper rings (6 stages), 128-deep K
// steps, 64-column tiles, four waves of 64 x 64 at 128 rows.
template <int EPI, int MBW, int JW, int WM, int WN, int D>
__global__ __launch_bounds__(64 * WM * WN) void gemm_rows_kernel(const Params p) {
  constexpr int NWV = WM * WN;                          // waves
  constexpr int KS = 64;                                // K step
  constexpr int TM = 32 * MBW * WM, TN = 32 * JW * WN;  // tile rows and columns
  constexpr int RB = KS * 2, CPR = RB / 16;             // bytes and 16-byte chunks of a tile row per step
  constexpr int RPL = 64 / CPR;                         // tile rows per 1 KB load
  constexpr int LA = TM * RB / 1024 / NWV, LW = TN * RB / 1024 / NWV;  // 1 KB loads per wave and stage
  constexpr int NL = LA + LW, STAGE = (TM + TN) * RB;
  static_assert(LA >= 1 && LW >= 1 && D >= 2 && (D - 2) * NL < 64, "loads in flight");
  static_assert(D * STAGE <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[D * STAGE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mt = (p.M + TM - 1) / TM;
  const int bid = blockIdx.x;
  if constexpr (is_logits(EPI)) {
    const int nwg = mt * ((p.N + TN - 1) / TN);
    if (bid >= nwg) return wide_rows(p, lane, NWV * (bid - nwg) + wave, NWV * (gridDim.x - nwg));
  }
  const int ks = bid % p.splitk, t = bid / p.splitk;
  const int m0 = (t % mt) * TM, n0 = (t / mt) * TN;
  const int K = p.K, nk_all = K / KS;
  const int k_begin = (int)((int64_t)nk_all * ks / p.splitk), k_end = (int)((int64_t)nk_all * (ks + 1) / p.splitk);
  const int nk = k_end - k_begin;

  // Load j of this wave fills the RPL tile rows RPL (NWV j + wave) ..; lane l writes
  // slot l % CPR of row l / CPR and fetches the chunk that belongs there.
  const int w_rows = EPI == kGemmSwiGLU ? (p.N >> 1) : p.N;
  const uint16_t* asrc[LA];
  const uint16_t* wsrc[LW];
  auto rswz = [](int r) { return (r & 7) ^ ((r >> 3) & 1); };
  auto chunk = [&](int r) { return ((lane & (CPR - 1)) ^ rswz(r)) * 8 + k_begin * KS; };
#pragma unroll
  for (int j = 0; j < LA; ++j) {
    const int r = RPL * (NWV * j + wave) + lane / CPR;
    asrc[j] = p.A + (int64_t)min(m0 + r, p.M - 1) * K + chunk(r);  // rows past M repeat the last; never stored
  }
#pragma unroll
  for (int j = 0; j < LW; ++j) {
    const int r = RPL * (NWV * j + wave) + lane / CPR;
    // SwiGLU: each 32-row block holds 16 gate rows, then the 16 up rows of the same outputs
    const int wr = EPI == kGemmSwiGLU ? (n0 >> 1) + 16 * (r >> 5) + (r & 15) : n0 + r;
    const uint16_t* wb = EPI == kGemmSwiGLU && (r & 16) ? p.W2 : p.W;
    wsrc[j] = wb + (int64_t)min(wr, w_rows - 1) * K + chunk(r);  // rows past N repeat the last; never stored
  }
  // The column tiles of an unsplit launch walk K from starts of their own, wrapping
  // around, as do those whose slices begin at multiples of 4 KB within a row: all
  // at the same offset of rows a power of two apart, they press on a few memory
  // channels at a time (8B-shaped gate/up over 32 rows: 50.9 -> 40.7 us, with the
  // weights loaded non-temporally; 64 rows 53.3 -> 44.2).  Row tiles of one column
  // tile share its start: they read the same weights at the same time, and every
  // row is summed in the same order.  Logits keep one order in every tile
  // (logits_kstride).
  const bool rotate = !is_logits(EPI) && (p.splitk == 1 || (nk * RB) % 4096 == 0);
  const int rot = rotate ? (int)(((unsigned)(t / mt) * 13u) % (unsigned)nk) : 0;
  auto issue = [&](int k) {
    uint8_t* st = smem + (k % D) * STAGE;
    const int kk = is_logits(EPI) ? (int)((unsigned)(k * p.kstride) % (unsigned)nk) : k + rot < nk ? k + rot : k + rot - nk;
#pragma unroll
    for (int j = 0; j < LA; ++j) {
      const uint16_t* src = asrc[j] + (int64_t)kk * KS;
      uint8_t* dst = st + 1024 * (NWV * j + wave);
      __builtin_amdgcn_global_load_lds(src, (lds_ptr)dst, 16, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < LW; ++j) {
      const uint16_t* src = wsrc[j] + (int64_t)kk * KS;
      uint8_t* dst = st + TM * RB + 1024 * (NWV * j + wave);
      __builtin_amdgcn_global_load_lds(src, (lds_ptr)dst, 16, 0, 2);  // non-temporal: read once
    }
  };

  constexpr int PA = parts_of(EPI);  // A blocks per accumulator block
  static_assert(MBW % PA == 0, "whole output blocks");
  Accum<EPI, MBW / PA, JW> sums;
  auto& acc = sums.acc;

  const int wm = wave / WN, wn = wave % WN;
  const int rl = lane & 31, kh = lane >> 5;
  int aoff[MBW], woff[JW];
#pragma unroll
  for (int i = 0; i < MBW; ++i) aoff[i] = (32 * (MBW * wm + i) + rl) * RB;
#pragma unroll
  for (int j = 0; j < JW; ++j) woff[j] = (TM + 32 * (JW * wn + j) + rl) * RB;
  const int f = rswz(rl);  // the row swizzle depends on the row's low four bits only

#pragma unroll
  for (int s = 0; s < D - 1; ++s)
    if (s < nk) issue(s);
  for (int k = 0; k < nk; ++k) {
    // step k has landed once only the later steps' loads are in flight
    const int later = nk - 1 - k;
    if (later >= D - 2) wait_vm<(D - 2) * NL>();
    else if (D > 3 && later == D - 3) wait_vm<(D > 3 ? D - 3 : 0) * NL>();
    else if (D > 4 && later == D - 4) wait_vm<(D > 4 ? D - 4 : 0) * NL>();
    else wait_vm<0>();
    // Every wave's loads of step k have landed, and every wave's reads of step
    // k - 1 have returned (their products were issued), so its stage takes step
    // k + D - 1.
    block_barrier();
    if (k + D - 1 < nk) issue(k + D - 1);
    const uint8_t* st = smem + (k % D) * STAGE;
#pragma unroll
    for (int s = 0; s < KS / 16; ++s) {
      const int c = ((2 * s + kh) ^ f) * 16;
      v4u fa[MBW], fw[JW];
#pragma unroll
      for (int j = 0; j < JW; ++j) fw[j] = *reinterpret_cast<const v4u*>(st + woff[j] + c);
#pragma unroll
      for (int i = 0; i < MBW; ++i) fa[i] = *reinterpret_cast<const v4u*>(st + aoff[i] + c);
      if (s == 0) sums.begin_step(p);  // while the fragments are on their way
#pragma unroll
      for (int i = 0; i < MBW; ++i)
#pragma unroll
        for (int j = 0; j < JW; ++j) acc[i / PA][j] = mfma32(fa[i], fw[j], acc[i / PA][j]);
    }
    wait_lds();  // no read of this step's stage is in flight past the next barrier
  }
  store_tile<EPI, MBW / PA, JW>(p, sums, lane, (m0 + 32 * MBW * wm) / PA, n0, JW * wn, ks);
}

}  // namespace

// ------------------------------------------------------------------ launch plan
// Workgroup tiles and the time of a 64-deep K step of one of them with a tile on
// every CU, measured over the projections of the 8B, 32B, 70B and Qwen3 shapes
// at 20 to 2048 rows (us; the step of a small tile is the wait for its weights).
struct Tile {
  int rows, cols;
  float step_us;
  bool few;  // at most 128 rows of A
};
static constexpr Tile kTiles[] = {
    {32, 128, 0.58f, true},   {64, 128, 0.64f, true},   {128, 128, 0.74f, true},
    {128, 256, 1.20f, true},  {128, 256, 1.12f, false}, {256, 128, 1.10f, false},
    {256, 160, 1.32f, false}, {256, 224, 1.65f, false}, {256, 256, 1.75f, false},
};
constexpr int kTileCount = sizeof(kTiles) / sizeof(kTiles[0]);

// Tiles built for an epilogue: the logits' two sets of sums leave no registers for one
// part of 256 x 160 and wider, and two parts of a row take two 32-row blocks of a wave.
constexpr bool has_tile(int epi, int t) {
  return epi == kGemmLogits ? t <= 5 : epi == kGemmLogitsSplit ? t >= 1 : true;
}

// The tile and K slices of least estimated time: whole rounds of the 256 CUs
// times a slice's K steps, 4 us for the launch, its first loads and its
// stores, and for each slice 8 bytes per value (a split product's slices are
// written here and read by the consumer, an unsplit one is added to the
// residual) at 5 TB/s.  At most eight slices (the consumers
// add no more), of at least four steps, and no more than part_elems holds.
// Over eighteen projections of the shapes above at eleven row counts from 20 to
// 2048 (198 products, two runs) the choice is the fastest of all tiles and slices or
// within 8% of it in 195 and 190, and 16% off at worst (8192 x 8192 at 20 rows);
// most of the misses are output and down projections at 200 rows, where the model
// favours one or two slices too many (5120 x 5120: 33.1 us against 30.4).
GemmPlan gemm_plan(int epi, int M, int N, int K, int64_t part_elems) {
  GemmPlan best{kTileCount - 1, 1};
  float best_us = 0.f;
  const int nk = K / BK;
  for (int t = 0; t < kTileCount; ++t) {
    const Tile& T = kTiles[t];
    if (T.few && M > 128) continue;
    if (T.rows == 128 && !T.few && M <= 128) continue;  // the few-row tile of this size streams better (108 against 116 us)
    if (!has_tile(epi, t)) continue;
    const int64_t tiles = (int64_t)((M + T.rows - 1) / T.rows) * ((N + T.cols - 1) / T.cols);
    for (int s = 1; s <= kGemmMaxSlices; ++s) {
      if (s > 1 && (s > nk / 4 || epi != kGemmPartialF32 || (int64_t)s * M * N > part_elems)) break;
      // 64 one-part accumulators a thread to fold (64 bf16 rows of the 8B head: 232 us, against 204 in tiles of 64 x 128)
      const float step_us = t == 3 && epi == kGemmLogits ? 1.2f * T.step_us : T.step_us;
      const float us = (float)((tiles * s + 255) / 256) * ((nk + s - 1) / s) * step_us + 4.f +
                       s * (float)M * N * 8e-6f / 5.f;
      if (best_us == 0.f || us < best_us) {
        best_us = us;
        best = GemmPlan{t, s};
      }
    }
  }
  return best;
}

template <int EPI>
static hipError_t launch_tile(const Params& p, int tile, hipStream_t s) {
  if (tile < 0 || tile >= kTileCount || !has_tile(EPI, tile)) return hipErrorInvalidValue;
  const Tile& T = kTiles[tile];
  const int64_t tiles = (int64_t)((p.M + T.rows - 1) / T.rows) * ((p.N + T.cols - 1) / T.cols) * p.splitk;
  const int wide = is_logits(EPI) ? min(kWideWorkgroups, (p.N + 4 * kWideCols - 1) / (4 * kWideCols)) : 0;  // wide_rows
  const dim3 grid((unsigned)(tiles + wide));
  switch (tile) {
    case 0:
      if constexpr (has_tile(EPI, 0)) hipLaunchKernelGGL((gemm_rows_kernel<EPI, 1, 1, 1, 4, 4>), grid, dim3(256), 0, s, p);
      break;
    case 1: hipLaunchKernelGGL((gemm_rows_kernel<EPI, 2, 1, 1, 4, 3>), grid, dim3(256), 0, s, p); break;
    case 2: hipLaunchKernelGGL((gemm_rows_kernel<EPI, 2, 1, 2, 4, 4>), grid, dim3(512), 0, s, p); break;
    case 3: hipLaunchKernelGGL((gemm_rows_kernel<EPI, 2, 2, 2, 4, 3>), grid, dim3(512), 0, s, p); break;
    case 4: hipLaunchKernelGGL((gemm_tile_kernel<EPI, 128, 8>), grid, dim3(64 * NW), 0, s, p); break;
    case 5: hipLaunchKernelGGL((gemm_tile_kernel<EPI, 256, 4>), grid, dim3(64 * NW), 0, s, p); break;
    case 6:
      if constexpr (has_tile(EPI, 6)) hipLaunchKernelGGL((gemm_tile_kernel<EPI, 256, 5>), grid, dim3(64 * NW), 0, s, p);
      break;
    case 7:
      if constexpr (has_tile(EPI, 7)) hipLaunchKernelGGL((gemm_tile_kernel<EPI, 256, 7>), grid, dim3(64 * NW), 0, s, p);
      break;
    case 8:
      if constexpr (has_tile(EPI, 8)) hipLaunchKernelGGL((gemm_tile_kernel<EPI, 256, 8>), grid, dim3(64 * NW), 0, s, p);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_gemm(int epi, const GemmPlan& plan, const uint16_t* A, const uint16_t* W, const uint16_t* W2, int M,
                       int N, int K, float* C, uint16_t* Cb, int* err_flag, hipStream_t s) {
  if (M <= 0 || N <= 0 || K <= 0 || K % BK || plan.slices < 1 || plan.slices > K / BK) return hipErrorInvalidValue;
  if (epi == kGemmSwiGLU && N % 32) return hipErrorInvalidValue;  // whole 16-output gate/up blocks
  // the nonlinearity and the residual update need complete sums: only the partial epilogue splits K
  if (epi != kGemmPartialF32 && plan.slices != 1) return hipErrorInvalidValue;
  const Params p{A, W, W2, M, N, K, plan.slices, C, Cb, err_flag, 0, nullptr, 1, 1, nullptr, 0, nullptr, nullptr};
  switch (epi) {
    case kGemmResidF32: return launch_tile<kGemmResidF32>(p, plan.tile, s);
    case kGemmSwiGLU: return launch_tile<kGemmSwiGLU>(p, plan.tile, s);
    case kGemmPartialF32: return launch_tile<kGemmPartialF32>(p, plan.tile, s);
    default: return hipErrorInvalidValue;
  }
}

// ------------------------------------------------------------------ logits of many rows
// The rows of a chunk as matrix operands.  Each row v (times the gain, where that is not
// folded into the matrix) is scaled by a power of two that brings its largest value
// into [2^13, 2^14).  A bf16 row without a gain is taken as fp16, exactly.  An fp32
// row is taken as an fp16 high part and the fp16 rounding of what is left: 22 to 23 bits
// of its values down to 2^-16 of the largest, and smaller ones to 2^-39 of it.  The
// error against 64-bit sums over the stored matrix is then that of the GEMV's fp32
// sums (1.2e-7 each, 8B head).  Rows of which that is not so, because the fp16 part of
// a bf16 row is not exact, more than an eighth of an fp32 row's values are
// that small or there is an infinity, are operands of zeros here and go through
// wide_rows.  Row r's factor is 1 / rms(v) and the power of two back, in 64
// bits (fp32 would not hold every such product, and its roundings, the same for a whole
// row, were half of the logits' error).  One workgroup per row; rows past `rows` fill their block with zeros.

struct HeadRow {  // a row of the head's input: values 4 k .. + 3, and these times the gain
  const void* in;
  int bf16;
  const uint16_t* gain;
  int64_t first;  // the row's first value / 4
  __device__ __forceinline__ f32x4 load(int k) const {
    if (bf16) {
      const uint2 e = reinterpret_cast<const uint2*>(in)[first + k];
      return f32x4{__uint_as_float(e.x << 16), __uint_as_float(e.x & 0xffff0000u), __uint_as_float(e.y << 16),
                   __uint_as_float(e.y & 0xffff0000u)};
    }
    return reinterpret_cast<const f32x4*>(in)[first + k];
  }
  __device__ __forceinline__ f32x4 gained(f32x4 v, int k) const {
    if (gain) {
      const uint2 g = reinterpret_cast<const uint2*>(gain)[k];
      v *= f32x4{__uint_as_float(g.x << 16), __uint_as_float(g.x & 0xffff0000u), __uint_as_float(g.y << 16),
                 __uint_as_float(g.y & 0xffff0000u)};
    }
    return v;
  }
};

template <int PARTS>
__global__ __launch_bounds__(256) void head_rows_kernel(const void* in, int in_bf16, const uint16_t* gain, int rows,
                                                        int H, float eps, uint16_t* a, double* row_scale, int* row_exp) {
  const int r = blockIdx.x, tid = threadIdx.x;
  uint2* hi = reinterpret_cast<uint2*>(a + (int64_t)(PARTS * (r & ~31) + (r & 31)) * H);
  uint2* lo = reinterpret_cast<uint2*>(a + (int64_t)(PARTS * (r & ~31) + 32 + (r & 31)) * H);
  auto zeros = [&] {
    for (int k = tid; k < H / 4; k += 256) {
      hi[k] = uint2{0u, 0u};
      if (PARTS == 2) lo[k] = uint2{0u, 0u};
    }
  };
  if (r >= rows) return zeros();
  const HeadRow row{in, in_bf16, gain, (int64_t)r * (H / 4)};
  double ss = 0.;
  float mx = 0.f;
  for (int k = tid; k < H / 4; k += 256) {
    const f32x4 v = row.load(k), w = row.gained(v, k);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ss = fma((double)v[i], (double)v[i], ss);
      mx = fmaxf(mx, fabsf(w[i]));
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    ss += __shfl_xor(ss, o);
    mx = fmaxf(mx, __shfl_xor(mx, o));
  }
  __shared__ double rs[4];
  __shared__ float rm[4];
  if ((tid & 63) == 0) {
    rs[tid >> 6] = ss;
    rm[tid >> 6] = mx;
  }
  __syncthreads();
  ss = (rs[0] + rs[1]) + (rs[2] + rs[3]);
  mx = fmaxf(fmaxf(rm[0], rm[1]), fmaxf(rm[2], rm[3]));
  // 2^e brings the row below 2^14; a row of zeros stays as it is.  Beside an infinity (a
  // value, or its product with the gain) the finite values are brought there from the
  // largest fp32 can hold.  A sum of squares beyond fp32 makes the factor 0, as the GEMV has it.
  const int e = mx == 0.f ? 0 : mx < INFINITY ? 13 - ilogbf(mx) : 13 - 127;
  bool wide = mx == INFINITY;
  if (!wide) {
    int lost = 0;  // values that the parts hold to fewer bits
    for (int k = tid; k < H / 4; k += 256) {
      const f32x4 w = row.gained(row.load(k), k);
      uint16_t h[4], l[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = ldexpf(w[i], e);
        const _Float16 vh = (_Float16)v;
        const float rest = v - (float)vh;
        h[i] = __builtin_bit_cast(uint16_t, vh);
        l[i] = __builtin_bit_cast(uint16_t, (_Float16)rest);
        lost += PARTS == 1 ? rest != 0.f : fabsf(v) < 0.25f && v != 0.f;
      }
      hi[k] = uint2{h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16)};
      if (PARTS == 2) lo[k] = uint2{l[0] | ((uint32_t)l[1] << 16), l[2] | ((uint32_t)l[3] << 16)};
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) lost += __shfl_xor(lost, o);
    __shared__ int rl[4];
    if ((tid & 63) == 0) rl[tid >> 6] = lost;
    __syncthreads();
    wide = rl[0] + rl[1] + rl[2] + rl[3] > (PARTS == 1 ? 0 : H / 8);
  }
  if (wide) zeros();
  if (tid == 0) {
    const double scale = fabs((float)ss == INFINITY ? 0. : ldexp(1.0 / sqrt(ss / H + (double)eps), -e));
    row_scale[r] = wide ? -scale : scale;
    row_exp[r] = e;
  }
}

// Order of the logits' K steps, the same in every tile and kernel: equal rows of
// the matrix then give equal logits wherever they lie (the lowest index of a tie
// is the caller's to find) and a row the same bits however many rows are asked
// for.  A stride of a quarter of the steps and one: the loads in flight spread
// over a row, where all workgroups in natural order press on a few memory
// channels (8B head, 5 and 64 fp32 rows, before sums were folded: 217 and 245 us in natural
// order, 175 and 204 so; 164 and 203 with a start of its own for each tile; strides of 5
// to 33 steps of the 64 were no faster than 17).
static int logits_kstride(int nk) {
  int s = nk > 4 ? nk / 4 + 1 : 1;
  auto gcd = [](int a, int b) {
    while (b) {
      const int r = a % b;
      a = b;
      b = r;
    }
    return a;
  };
  while (gcd(s, nk) != 1) ++s;
  return s;
}

// K steps that an accumulator of the logits runs over: as many as leave the error at the
// GEMV's (K = 4096: fp32 rows 1.2e-7 each, and 1.1e-7 with one step; bf16 rows
// 0.8e-7 against 1.0e-7; K = 320, fp32 rows: 1.0e-7 each with one step, 1.2e-7 with two).
// Each fold costs 3 vector instructions a value: 256 fp32 rows of the 8B head 521 us
// without folds, 560 with one every two steps, 660 with one every step.
static int logits_fold(int parts, int nk) { return parts == 2 && nk < 32 ? 1 : 2; }

hipError_t launch_head_logits(const void* in, int in_bf16, const uint16_t* gain, const uint16_t* w, int rows, int N,
                              int K, float eps, uint16_t* a, double* row_scale, float* logits, int* err_flag,
                              hipStream_t s, int tile) {
  const int parts = in_bf16 && !gain ? 1 : 2;
  if (rows <= 0 || rows > kHeadChunk * 2 / parts || N <= 0 || K <= 0 || K % BK) return hipErrorInvalidValue;
  int* row_exp = reinterpret_cast<int*>(row_scale + 2 * kHeadChunk);
  const int blocks = (rows + 31) / 32, epi = parts == 1 ? kGemmLogits : kGemmLogitsSplit;
  if (parts == 1)
    hipLaunchKernelGGL(head_rows_kernel<1>, dim3(32 * blocks), dim3(256), 0, s, in, in_bf16, gain, rows, K, eps, a,
                       row_scale, row_exp);
  else
    hipLaunchKernelGGL(head_rows_kernel<2>, dim3(32 * blocks), dim3(256), 0, s, in, in_bf16, gain, rows, K, eps, a,
                       row_scale, row_exp);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int M = 32 * blocks * parts;
  const Params p{a, w, nullptr, M, N, K, 1, logits, nullptr, err_flag, rows, row_scale, logits_kstride(K / BK),
                 logits_fold(parts, K / BK), in, in_bf16, gain, row_exp};
  if (tile < 0) tile = gemm_plan(epi, M, N, K, 0).tile;
  return parts == 1 ? launch_tile<kGemmLogits>(p, tile, s) : launch_tile<kGemmLogitsSplit>(p, tile, s);
}

}  // namespace kf
