// Device-side definitions shared by the translation units of the absorbed-MLA decode library: tile and
// layout constants, the kernel parameter block, and the small helpers every decode kernel uses (guarded
// exponent add of Lemma 3.1, bf16 packing, the direct-to-LDS tile loads).
#ifndef AMLA_DEVICE_H_
#define AMLA_DEVICE_H_

#include <stdint.h>

#include "amla_plan.h"

constexpr int kDqk = 576;
constexpr int kDv = 512;
constexpr int kBlock = 64;               // keys per cache block
constexpr int kRowBytes = kDqk * 2;      // 1152 bytes of bf16 per cached row
constexpr int kLdsRow = kRowBytes + 16;  // padded LDS row: 73 chunks of 16 B (odd -> no bank conflicts)
constexpr int kChunksPerRow = kLdsRow / 16;           // 73
constexpr int kTileBytes = kBlock * kLdsRow;          // 74752 = 73 * 1024
constexpr int kTileLoads = kTileBytes / 1024;         // 73 wave-wide 1 KiB direct-to-LDS loads
constexpr int kRowsPerWg = 128;
constexpr int kThreads = 256;
constexpr int kFewRows = 32;             // sequences of at most so many rows have kernels of their own
constexpr int kLdsBytes = 2 * kTileBytes;             // double buffer, 149504 B of the 160 KiB

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4;
typedef __attribute__((__vector_size__(2 * sizeof(int)))) int i32x2;

// Target hooks.  The definitions below are the gfx950 ones; a CPU build of these kernels (tests
// only: bounds-checked runs of the index logic) defines them beforehand.
#ifndef AMLA_TARGET_HOOKS
#define LDS_PTR(T) __attribute__((address_space(3))) T*
#define GLB_PTR(T) __attribute__((address_space(1))) T*
// every direct-to-LDS load of this wave has landed
#define AMLA_WAIT_TILE_LOADS() asm volatile("s_waitcnt vmcnt(0)" ::: "memory")
// make x opaque to the optimiser at this point (stops hoisting of what is derived from it)
#define AMLA_OPAQUE(x) asm volatile("" : "+v"(x))
// one wave per SIMD: the whole 512-register file belongs to it
#define AMLA_ONE_WAVE_PER_SIMD __attribute__((amdgpu_waves_per_eu(1, 1)))
// One 16-byte-per-lane direct-to-LDS load (lane l lands at lds + 16 l, lds wave-uniform) issued from inline
// assembly, so that the compiler's wait-count pass does not know LDS is being written: it otherwise puts a
// full vmcnt(0) in front of the first transposing LDS read that follows, and the second product could never
// overlap the loads.  The kernels' own wait (AMLA_WAIT_TILE_LOADS, then the barrier) is what orders the tile's
// arrival before its readers.  The compiler's waits for its own vector-memory operations stay correct with
// loads it does not count: the counter is in-order and extra outstanding operations only make a wait longer.
#define AMLA_HIDDEN_LDS_LOAD(gptr, lds)                                                                      \
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"                              \
               :                                                                                             \
               : "v"(gptr), "s"(__builtin_amdgcn_readfirstlane((unsigned)(__UINTPTR_TYPE__)(lds)))           \
               : "memory", "m0")
// a use of x the compiler must honour here: whatever load produces x is waited for at this point
#define AMLA_ARRIVED(x) asm volatile("" : : "v"(x))
// element i of an int32 array that no kernel writes while this one runs, read through the scalar cache
// when i is wave-uniform (a load that counts in lgkmcnt, not in the vmcnt of the tile loads)
#define AMLA_UNIFORM_LOAD_I32(p, i) (((const __attribute__((address_space(4))) int32_t*)(uintptr_t)(p))[i])
#endif

struct DecodeParams {
  const uint16_t* q;        // [B, G, 576] bf16 bits (G = s_q * H rows per sequence)
  const uint16_t* kv;       // [num_blocks, 64, 576]
  const int32_t* table;     // [B, max_blocks]
  const int32_t* seqlens;   // [B]
  uint16_t* out;            // [B, G, 512] bf16 bits
  float* lse;               // [B, G] or null
  float* part_o;            // [n_splits, B, G, 512] (n_splits > 1); FP16 rows from the row-rescale kernels, else FP32
  float* part_lse;          // [n_splits, B, G]
  float scale_log2e;        // softmax_scale * log2(e)
  int32_t batch;
  int32_t rows;             // G
  int32_t n_tiles;          // ceil(G / rows of a workgroup)
  int32_t n_splits;
  int32_t max_blocks;
  int32_t n_streams;        // batch * n_splits; balanced decomposition: number of workers
  int32_t flags;
  int32_t num_blocks;       // physical blocks in the pool (the balanced kernel clamps table entries)
  int32_t heads;            // rows of a sequence are (t, h) flattened: t * heads + h
  int32_t causal_span;      // s_q - 1 under the causal mask among the s_q query tokens, else 0
  int32_t s_q;              // query tokens per sequence in the q array
  const int32_t* q_lens;    // [B] query tokens sequence b really has (<= s_q), or null: s_q everywhere
  int32_t* plan;            // balanced, row-rescale kernels: what the merge has to know of the plan (PlanUnits), in the workspace
  int32_t tile_workers;     // balanced: workers where row tiles are items of the plan of their own (PlanUnits); 0: they are not in this call
  int32_t tile_shift;       // log2 of a workgroup's rows
  int32_t even_xcds;        // equal shares, row-rescale kernels: every XCD an equal stretch of the workgroups, else whole sequences in turn
  int32_t early_queries;    // equal shares, tiles of 128 rows: query rows are asked for before a share is known to have blocks (QueryLoads)
};

// A row's shift that puts its limit before every key: the row of a padding token.
constexpr int kNoKeys = 1 << 30;

// Lemma 3.1 with a guard: x * 2^delta as an integer add of n23 = delta << 23 (delta <= 0) on the
// bit pattern.  The saturating add pins a negative float whose exponent would go below zero at
// 0x80000000 (-0.0); the max with the sign bit turns a wrapped positive float into +0.0.
// n23 may also carry a small mantissa term of either sign (Algorithm 2's eps inside N): the guard
// only concerns sums that leave the float's own sign range.
__device__ __forceinline__ float exponent_add(float x, int n23) {
  const int i = __float_as_int(x);
  int r = __builtin_elementwise_add_sat(i, n23);
  r = max(r, i & (int)0x80000000);
  return __int_as_float(r);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {
  f32x2 v = {lo, hi};
  bf16x2 b = __builtin_convertvector(v, bf16x2);   // round to nearest even
  return __builtin_bit_cast(unsigned, b);
}

// two FP32 values as a pair of FP16 (round to nearest even), lo in the low half
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ unsigned pack_f16(float lo, float hi) {
  f32x2 v = {lo, hi};
  f16x2 b = __builtin_convertvector(v, f16x2);
  return __builtin_bit_cast(unsigned, b);
}

// Issue this wave's share (one of NWAVES) of the direct-to-LDS loads of one 64 x 576 bf16 block.
// LDS destination of load i is the 1 KiB range [i * 1024, (i + 1) * 1024) of the tile buffer,
// lane l landing at + 16 l; chunk c = 64 i + l of the padded tile is row c / 73, column chunk
// c % 73, the 73rd chunk of a row being padding (it receives 16 harmless bytes).
template <int NWAVES = 4, bool HIDDEN = false>
__device__ __forceinline__ void issue_tile_loads(const uint8_t* block_base, LDS_PTR(uint8_t) buf,
                                                 int wave, int lane) {
  // keep the per-lane offsets out of loop-invariant hoisting: 19 of them per lane would
  // cost more registers than recomputing them costs VALU slots
  AMLA_OPAQUE(lane);
#pragma unroll
  for (int k = 0; k < (kTileLoads + NWAVES - 1) / NWAVES; ++k) {
    const int i = wave + NWAVES * k;
    if (i < kTileLoads) {
      const int c = i * 64 + lane;
      const int row = (int)(((unsigned)c * 57457u) >> 22);      // c / 73 for c < 4672
      const int cc = c - row * kChunksPerRow;
      const int off = (cc < kChunksPerRow - 1) ? (c - row) * 16 : 0;
      if (HIDDEN) {
        AMLA_HIDDEN_LDS_LOAD(block_base + off, buf + i * 1024);
      } else {
        __builtin_amdgcn_global_load_lds((const GLB_PTR(void))(block_base + off),
                                         (LDS_PTR(void))(buf + i * 1024), 16, 0, 0);
      }
    }
  }
}

constexpr float kLazyThreshold = 8.f;   // base-2 units: the weights may grow to 2^8 before the reference moves

__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}

__device__ __forceinline__ int wave_inclusive_scan(int v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o);
    if (lane >= o) v += u;
  }
  return v;
}

// v <- the sum of v over the wave, in every lane.  On the vector unit's lane shifts: six dependent shuffles through LDS
// are about 700 cycles, and this stands before a workgroup's first load.
#ifndef AMLA_TARGET_HOOKS
template <int CTRL, int ROWS>
__device__ __forceinline__ int lane_shift(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, true); }
#define AMLA_WAVE_SUM(v)                                                                         \
  do {                                                                                           \
    v += lane_shift<0x111, 0xf>(v); /* row_shr 1, 2, 4, 8: lane 15 of a row has the row's */     \
    v += lane_shift<0x112, 0xf>(v);                                                              \
    v += lane_shift<0x114, 0xf>(v);                                                              \
    v += lane_shift<0x118, 0xf>(v);                                                              \
    v += lane_shift<0x142, 0xa>(v); /* row_bcast 15 into rows 1 and 3 */                         \
    v += lane_shift<0x143, 0xc>(v); /* row_bcast 31 into rows 2 and 3: lane 63 has them all */   \
    v = __builtin_amdgcn_readlane(v, 63);                                                        \
  } while (0)
#else
#define AMLA_WAVE_SUM(v)                                    \
  do {                                                      \
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o); \
  } while (0)
#endif

// What the balanced decomposition lays end to end and cuts, the units of its plan: the cache blocks of all sequences, each range of them worked by a
// workgroup for every row tile; or, where sequences have different numbers of tokens, the blocks of all (sequence, row tile) items whose tile has
// rows of real tokens, tile by tile, each range worked by one workgroup.  The second leaves no workgroup with padding tiles, but the tiles of a
// sequence no longer share its blocks in an XCD's L2, and more results are merged.  So it is taken where a quarter of the (tile, block) pairs at
// least are padding and the workers' ranges are long enough for that; every workgroup decides alike.
//   Tiles of 128 rows: ranges are shorter by 0.6 blocks and 0.05 for every further piece that an item then has in the merge.  us a call (ADD), by sequence / by
// tile: 40 sequences of 130 .. 5000 keys, three tokens, 2/3 of the pairs real 109.2 / 104.7, all of them 113.6 / 135.0; 64 of 3000 .. 4000, four, 5/8 real
// 244.9 / 188.7; 100 of 100 .. 2000, two, 3/4 real 107.6 / 102.8; 17 of four, one real 189.9 / 90.1; 2 of three, one real, 85 more pieces for 2.7 blocks 42.6 /
// 51.5.  Of 743 shapes of 1 .. 256 sequences, two to four row tiles and 3 .. 500 blocks 285 take it: 1.21 times as fast, seven of them more than 3 % slower (at
// worst 40.3 / 46.5 and 85 / 97; 17 of three tokens and 24 blocks each 48.9 / 53.5, ADD_COMP: ranges by sequence end where the sequences do).
//   Tiles of 16 and 32 rows: ranges are shorter by a block and a half.  (The blocks and the merge take half as long, and no more workgroups than one round
// holds are there to fill.)  60 sequences of two tokens of 64 heads, one real, 32.3 / 27.3; 3 of four of 128, up to two real, 30.8 / 23.1; 7 of three, two
// real, 32.1 / 35.4.  Of 300 shapes 60 take it: 1.06 times as fast.
//
// The merge reads who met which item from the workspace: note[0] = whether the plan went by row tiles, and from [1] on two for each
// (sequence, row tile of a workgroup): the worker that had its first block and the one that had its last.  (Worked out from the
// lengths again, by a wave for every one or two rows, the last of the calls above took 99.0 us and not 96.2.)
struct PlanUnits {
  const int32_t* seqlens;
  const int32_t* q_lens;   // null where no plan goes by tile
  int batch, max_blocks, s_q, heads, tile_shift;
  // row tiles with rows of real tokens
  __device__ __forceinline__ int live_tiles(const int q_len) const {
    return (int)(((unsigned)(min(max(q_len, 0), s_q) * heads) + (1u << tile_shift) - 1) >> tile_shift);
  }
};

// The balanced merges' arguments beside the rows.
struct MergePlan {
  PlanUnits units;
  const int32_t* note;   // DecodeParams::plan
  int rows, workers, n_tiles;
};

// Blocks of all sequences, units by tile too where `by_tile`, and this lane's part of the blocks before sequence b (AMLA_WAVE_SUM has the sum).  Kept to a
// few instructions: this stands before a workgroup's first load.
struct BatchUnits {
  int blocks, tiled, before;
};
__device__ __forceinline__ BatchUnits batch_units(const PlanUnits& u, const bool by_tile, int b, int lane) {
  BatchUnits s = {0, 0, 0};
  const int most = plan_len(0x7fffffff, u.max_blocks, kBlock);
  constexpr int kAhead = 4;   // 256 lengths in one round trip
  for (int c = 0; c < u.batch; c += 64 * kAhead) {
    int len[kAhead], tokens[kAhead];
    auto load = [&](const int32_t* from, int k) { return c + 64 * k < u.batch && c + 64 * k + lane < u.batch ? from[c + 64 * k + lane] : 0; };
#pragma unroll
    for (int k = 0; k < kAhead; ++k) len[k] = load(u.seqlens, k);
    if (by_tile)
#pragma unroll
      for (int k = 0; k < kAhead; ++k) tokens[k] = load(u.q_lens, k);
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      if (c + 64 * k >= u.batch) break;
      const int n = (int)(((unsigned)min(max(len[k], 0), most) + (kBlock - 1)) / kBlock);
      s.blocks += n;
      if (by_tile) s.tiled += n * u.live_tiles(tokens[k]);
      s.before += c + 64 * k + lane < b ? n : 0;
    }
  }
  AMLA_WAVE_SUM(s.blocks);
  if (by_tile) AMLA_WAVE_SUM(s.tiled);
  return s;
}

// Kernels defined in other translation units of the library, looked up by amla_decode.
typedef void (*AmlaDecodeKernel)(const DecodeParams);
AmlaDecodeKernel amla_row_rescale_kernel(int variant, bool balanced, bool iteration_512, int tile_rows, bool by_tile);   // amla_decode_rg.hip
int amla_row_rescale_lds_bytes();

#endif  // AMLA_DEVICE_H_
