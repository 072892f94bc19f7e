// HIP kernels and C ABI of libsbw (declared in include/sbw.h) for MI355X / gfx950.
//
// watermark   one streaming pass over the logits: each lane owns 16-byte vectors
//             of a row (4 fp32 or 8 bf16 logits; self-salt 4 of either), loads them,
//             derives the green decision in registers (seed, Philox4x32-10 draw, threshold
//             compare) and stores them back.  Row-uniform values (the window of previous
//             tokens, the context seed, key * J(p_i)) sit in scalar registers.
//             Context seeding shares one Philox block between the 4 tokens of a
//             counter; self-salt needs one block per token, and its workgroups take
//             several rows in turn with each candidate's hash and self term computed
//             once.  Launches that leave the chip mostly idle take one token per
//             lane instead.  Large self-salt launches (window of one token) instead draw each
//             column's self-term block once per slab of 12, 8 or 6 rows and queue in
//             LDS only the pairs whose row term is the smaller one (about half).
// argmax      greedy decoding of the watermarked logits without writing them: one
//             read of each logit, a per-segment (value, index) partial, a read-out
//             kernel per row.  Colours are drawn only for logits that can still
//             reach the segment's maximum.  Rows of a few hundred tokens: every
//             token scored, the winner stored, in one launch.
// candidates  the watermark restricted to caller-given candidate ids per row (the
//             top-k self-salt scheme): one workgroup per row.
// green_mask  one lane per 32-token word of the bit set.
// detect      one wavefront per sequence, or up to 16 wavefronts and several workgroups
//             for few sequences; each lane scores positions i, i+64, ... and a wave
//             counts green positions with a ballot + popcount.  With
//             repeated n-grams scored once: one workgroup per sequence and an LDS
//             hash set of first occurrences.
//
// The context window: row b of a watermark call sees the `width` tokens
// context[b*width .. b*width+width-1] (the tokens before the step); position i of a
// detected sequence sees tokens i-width .. i-1.  Width 1 is the previous token.
#include <hip/hip_runtime.h>
#include <float.h>
#include <math.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "sbw.h"
#include "sbw_device.hpp"

namespace sbw {
namespace {

// Launch-shape tuning knobs (compile-time; the defaults are the measured best).
#ifndef SBW_CONTEXT_UNROLL
#define SBW_CONTEXT_UNROLL 2   // 16-byte vectors per lane, context seeding (HBM-bound)
#endif
#ifndef SBW_CONTEXT_UNROLL_BF16
#define SBW_CONTEXT_UNROLL_BF16 2
#endif
// Self-salt, width 1: the split-term slab kernel.  12-row slabs when that makes at least
// SBW_SLAB12_MIN_GROUPS workgroups, else with 8-row, else (fp32) with 6-row slabs when that
// makes at least SBW_SLAB_MIN_GROUPS, bf16 SBW_SLAB_BF16_MIN_GROUPS (below that its
// long-lived waves leave the chip underfilled and the row kernel is faster).  12-row slabs
// need more workgroups than the others: with fewer than ~1.7 rounds of the ~1800 that fit at
// once, the last round's tail costs more than the shorter slabs' extra self terms.  bf16 us,
// slabs / row kernel: 12 rows, B = 700 of 152064 (4425 workgroups) 152 / 164, B = 512 (3225)
// 117.1 / 118.2; 8 rows, B = 400 (3750) 89.1 / 91.6, B = 300 (2850) 69.1 / 72.3, B = 280 (2625)
// 67.2 / 65.9, B = 256 (2400) 61.9 / 60.6.
// Context seeding: launches of at least SBW_XCD_ROWS_MIN rows (a multiple of 8) and
// SBW_XCD_ROWS_MIN_BYTES of logits, more than the 256 MB Infinity Cache holds, give
// each XCD whole rows (fp32 B = 512 / 1024 of 152064: 1 / 3 % faster, bf16 B = 1024:
// 3 %; B = 256 even, B = 128 and bf16 B = 512 of 128256 up to 1 % slower).
#ifndef SBW_XCD_ROWS_MIN
#define SBW_XCD_ROWS_MIN 512
#endif
#ifndef SBW_XCD_ROWS_MIN_BYTES
#define SBW_XCD_ROWS_MIN_BYTES (int64_t{256} << 20)
#endif
#ifndef SBW_SLAB_MIN_GROUPS
#define SBW_SLAB_MIN_GROUPS 2000
#endif
#ifndef SBW_SLAB_BF16_MIN_GROUPS
#define SBW_SLAB_BF16_MIN_GROUPS 2700
#endif
#ifndef SBW_SLAB12_MIN_GROUPS
#define SBW_SLAB12_MIN_GROUPS 3000
#endif

constexpr int kThreads = 256;            // 4 wavefronts of 64
constexpr int kMaxWidth = 8;             // longest context window
constexpr int kMidWidth = 4;             // windows of 2-4 (the paper's 4): own instantiations
constexpr int64_t kMaxGrid = 1ll << 20;  // blocks; grid-stride loops cover the rest
constexpr int64_t kMaxGridY = 65535;
constexpr int64_t kMaxEdgeY = 4096;      // grid rows of edge columns; a loop covers the rest

// Native vector types (the non-temporal builtins take these, not HIP's float4/uint4).
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A 16-byte vector of logits: 4 fp32 (as values) or 8 bf16 (as packed bits), and the same
// in memory, where it is aligned to one logit only: a row may start anywhere (an odd
// vocabulary, a slice of a padded buffer).  gfx950 takes 16-byte global accesses at any
// byte address, so both give the same instruction; what an odd address costs is a ninth
// 128-byte line for every 1 KB a wave moves.  Context pass, 256 rows of 152064 / 152065
// columns: fp32 48.1 / 51.9 us, bf16 26.2 / 27.4 us; the element-wise kernel that such
// rows took before: 117.7 and 102.9 us.
typedef f32x4 f32x4_memory __attribute__((aligned(4)));
typedef u32x4 u32x4_memory __attribute__((aligned(2)));
template <typename T>
struct VecOf {
  typedef f32x4 Value;
  typedef f32x4_memory Memory;
};
template <>
struct VecOf<uint16_t> {
  typedef u32x4 Value;
  typedef u32x4_memory Memory;
};

// The 4 tokens of one Philox counter: 16 bytes of fp32 logits, 8 of bf16.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef u32x2 u32x2_memory __attribute__((aligned(2)));
template <typename T>
struct QuadOf {
  typedef f32x4 Value;
  typedef f32x4_memory Memory;
};
template <>
struct QuadOf<uint16_t> {
  typedef u32x2 Value;
  typedef u32x2_memory Memory;
};

// Overloads, not a template: a template argument would lose the alignment.
__device__ __forceinline__ f32x4 stream_load(const f32x4_memory* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ u32x4 stream_load(const u32x4_memory* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ void stream_store(f32x4_memory* p, f32x4 v) { __builtin_nontemporal_store(v, p); }
__device__ __forceinline__ void stream_store(u32x4_memory* p, u32x4 v) { __builtin_nontemporal_store(v, p); }

__device__ __forceinline__ u32x2 stream_load(const u32x2_memory* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ void stream_store(u32x2_memory* p, u32x2 v) { __builtin_nontemporal_store(v, p); }

// How a row of V columns with token ids from vbase falls into 16-byte vectors whose first
// token id is a multiple of their kPer tokens (so that they hold whole Philox blocks):
// `head` columns before the first vector (0-3 fp32, 0-7 bf16; 0 unless the row is a shard
// starting at an odd id), `full` vectors, `tail` columns after the last.
struct RowSplit {
  uint32_t head, full, tail;
  uint32_t id;   // the first vector's token id / kPer
  __device__ __forceinline__ uint32_t edges() const { return head + tail; }
  // the column of edge e, 0 <= e < edges()
  template <uint32_t kPer>
  __device__ __forceinline__ uint32_t edge(uint32_t e) const {
    return e < head ? e : full * kPer + e;
  }
};
template <uint32_t kPer>
__host__ __device__ __forceinline__ RowSplit row_split(uint32_t V, uint32_t vbase) {
  const uint32_t to_block = (kPer - vbase % kPer) % kPer;
  const uint32_t head = to_block < V ? to_block : V;
  return RowSplit{head, (V - head) / kPer, (V - head) % kPer, (vbase + head) / kPer};
}
// ---------------------------------------------------------------------------
// Seeds.  kW is the compile-time bound on the window width: 1 for the
// previous-token path, kMaxWidth for wider windows (runtime width <= kW).
// ---------------------------------------------------------------------------
template <int kW>
struct RowSeed {
  uint64_t key;        // the watermark key
  uint64_t seed;       // context seeding: key * (sum of the window)
  uint64_t kjp[kW];    // self-salt: key * J(p_i) for the window tokens
  int width;
};

template <int kSeeding, int kW>
__device__ __forceinline__ RowSeed<kW> row_seed(uint64_t key, const int32_t* window, int width) {
  RowSeed<kW> rs;
  rs.key = key;
  rs.width = width;
  rs.seed = 0u;
  if (kSeeding == kContext) {
    uint64_t sum = 0u;
    for (int i = 0; i < (kW == 1 ? 1 : width); ++i) sum += static_cast<uint32_t>(window[i]);
    rs.seed = key * sum;
  } else {
#pragma unroll
    for (int i = 0; i < kW; ++i)
      rs.kjp[i] = (kW == 1 || i < width)
                      ? key * static_cast<uint64_t>(jenkins32(static_cast<uint32_t>(window[i])))
                      : 0u;
  }
  return rs;
}

// Self-salt seed of candidate v: the minimum over the window and v itself of
// key*J(w)*J(v).  Split in two: the candidate's terms J(v) and key*J(v)*J(v), which
// do not depend on the row, then the row's minimum.
struct CandTerm {
  uint32_t jv;     // J(v)
  uint64_t self;   // key * J(v) * J(v)
};

__device__ __forceinline__ CandTerm cand_term(uint64_t key, uint32_t v) {
  const uint32_t jv = jenkins32(v);
  return CandTerm{jv, mul_64x64(key, wide_mul(jv, jv))};
}

// The self-salt seed of a candidate from its terms and the row's key*J(p_i).
template <int kW>
__device__ __forceinline__ uint64_t self_salt_seed_t(const RowSeed<kW>& rs, const CandTerm& t) {
  uint64_t best = t.self;
#pragma unroll
  for (int i = 0; i < kW; ++i) {
    if (kW == 1 || i < rs.width) {
      const uint64_t x = lane_mul_64x32(rs.kjp[i], t.jv);
      best = x < best ? x : best;
    }
  }
  return best;
}

template <int kW>
__device__ __forceinline__ uint64_t self_salt_seed_w(const RowSeed<kW>& rs, uint32_t v) {
  return self_salt_seed_t(rs, cand_term(rs.key, v));
}

template <int kSeeding, int kW>
__device__ __forceinline__ uint32_t draw(const RowSeed<kW>& rs, uint32_t v) {
  if (kSeeding == kContext) return cbrng(v, rs.seed);
  return cbrng(v, self_salt_seed_w(rs, v));
}

// ---------------------------------------------------------------------------
// Context-seeded watermark vectors: one row seed, so the tokens of a Philox block
// share it.  fp32: a vector is the 4 tokens 4j..4j+3, exactly the 4 words of the
// block at counter j.  bf16: the 8 tokens 8j..8j+7 = blocks 2j and 2j+1.
// ---------------------------------------------------------------------------
__device__ __forceinline__ f32x4 bias_vec_context(f32x4 l, uint32_t j, uint64_t seed, uint32_t tm1,
                                                  float delta) {
  const Block blk = philox_block(j, key_of(seed));
  f32x4 o;
  o.x = bias_f32(l.x, delta, is_green(blk.w0, tm1));
  o.y = bias_f32(l.y, delta, is_green(blk.w1, tm1));
  o.z = bias_f32(l.z, delta, is_green(blk.w2, tm1));
  o.w = bias_f32(l.w, delta, is_green(blk.w3, tm1));
  return o;
}

__device__ __forceinline__ u32x4 bias_vec_context(u32x4 raw, uint32_t j, uint64_t seed, uint32_t tm1,
                                                  float delta) {
  const Key k = key_of(seed);
  const Block a = philox_block(2u * j, k);
  const Block b = philox_block(2u * j + 1u, k);
  const uint32_t x[8] = {a.w0, a.w1, a.w2, a.w3, b.w0, b.w1, b.w2, b.w3};
  const uint32_t in[4] = {raw.x, raw.y, raw.z, raw.w};
  uint32_t out[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    out[q] = bias_bf16x2(in[q], delta, is_green(x[2 * q], tm1), is_green(x[2 * q + 1], tm1));
  return u32x4{out[0], out[1], out[2], out[3]};
}

// One element of either dtype (columns outside whole vectors).
__device__ __forceinline__ float bias_elem(float l, float d, bool g) { return bias_f32(l, d, g); }
__device__ __forceinline__ uint16_t bias_elem(uint16_t l, float d, bool g) {
  return bias_bf16(l, d, g);
}

// The columns outside whole vectors (RowSplit), one lane a column, 16 rows a workgroup, in
// grid rows of their own.  A path of its own, so that the tiles' path keeps no registers for
// it (inside the tiles it cost 2-13 VGPRs a lane and with them a wave per SIMD: bf16 self-salt
// 256 x 152064, width 4, 96 -> 106 us), and only as many workgroups as have work: a column of
// one per row, most of them empty, cost their dispatch (1000 x 2001 fp32, self-salt: 9.5 us,
// 6.6 so; 500 x 32001 bf16, 32.0, 28.4).  They are a launch's grid rows from `slots` on, behind
// the tiles, which they delay in front (48 x 128259 bf16, self-salt: 14.3 us, 13.3 behind) and
// between (16.7); only context launches of many rows, bound by memory, spread them between the
// tiles, every 2^shift-th grid row (353 x 30079 bf16: 9.9 us behind, 9.5 spread; 500 x 32001
// 13.4 / 12.8; but 48 x 128259 6.5 / 6.75, 200 x 50257 9.0 / 9.1).
constexpr int64_t kSpreadRows = 300;
constexpr uint32_t kEdgeRows = 16;
static_assert(kThreads / kEdgeRows >= 14, "a row has at most 7 + 7 such columns");
template <typename T, int kSeeding, int kW, uint32_t kPer>
__device__ __forceinline__ void watermark_edges(T* logits, int64_t row_stride, const RowSplit& sp,
                                                int64_t B, const int32_t* context, int width,
                                                uint64_t key, uint32_t tm1, float delta,
                                                uint32_t vbase, uint32_t edge_row,
                                                uint32_t edge_rows) {
  const int64_t slot = static_cast<int64_t>(edge_row) * gridDim.x + blockIdx.x;
  const uint32_t e = threadIdx.x % (kThreads / kEdgeRows);
  if (e >= sp.edges()) return;
  for (int64_t row = slot * kEdgeRows + threadIdx.x / (kThreads / kEdgeRows); row < B;
       row += static_cast<int64_t>(edge_rows) * gridDim.x * kEdgeRows) {
    // the logit is on its way while the window is read and the colour drawn
    T* p = logits + row * row_stride + sp.edge<kPer>(e);
    const T l = *p;
    const RowSeed<kW> rs = row_seed<kSeeding, kW>(key, context + row * width, width);
    *p = bias_elem(l, delta, is_green(draw<kSeeding>(rs, vbase + sp.edge<kPer>(e)), tm1));
  }
}

// Context-seeded watermark.  Grid: x = tile of kThreads * kU vectors within a row, y = row
// (grid-stride over rows beyond the `slots` of the tiles), then grid rows for the edge columns;
// kSpread: every 2^slots-th grid row.
// Each lane issues its logits load before reading the row's window, so the scalar loads of
// the window overlap the HBM stream.  With xcd_rows (one row per y, B a multiple of 8) the
// workgroups are renumbered so that each of the 8 XCDs, which take workgroups in turn,
// streams whole rows: workgroup n goes to row 8 * (n / 8 / tiles) + n % 8, tile n / 8 % tiles.
template <typename T, int kU, int kW, bool kSpread>
__global__ void __launch_bounds__(kThreads)
watermark_vec_kernel(T* __restrict__ logits, int64_t row_stride, uint32_t V, int64_t B,
                     const int32_t* __restrict__ context, int width, uint64_t key, uint32_t tm1,
                     float delta, uint32_t vbase, uint32_t xcd_rows, uint32_t slots) {
  using VecT = typename VecOf<T>::Value;
  using MemT = typename VecOf<T>::Memory;
  constexpr uint32_t kPer = 16u / sizeof(T);  // elements per 16-byte vector
  const RowSplit sp = row_split<kPer>(V, vbase);
  const uint32_t full = sp.full;
  const uint32_t jbase = sp.id;
  if (kSpread ? ((blockIdx.y + 1u) & ((1u << slots) - 1u)) == 0u : blockIdx.y >= slots) {
    watermark_edges<T, kContext, kW, kPer>(logits, row_stride, sp, B, context, width, key, tm1, delta, vbase,
                                           kSpread ? blockIdx.y >> slots : blockIdx.y - slots,
                                           kSpread ? gridDim.y >> slots : gridDim.y - slots);
    return;
  }
  const uint32_t y = kSpread ? blockIdx.y - (blockIdx.y >> slots) : blockIdx.y;   // among the tiles' rows
  uint32_t first = blockIdx.x * (kThreads * kU);
  int64_t row0 = y;
  if (xcd_rows != 0u) {
    const uint32_t n = y * gridDim.x + blockIdx.x;
    const uint32_t q = n >> 3;
    row0 = static_cast<int64_t>(q / gridDim.x) * 8 + (n & 7u);
    first = (q % gridDim.x) * (kThreads * kU);
  }
  for (int64_t row = row0; row < B; row += kSpread ? gridDim.y - (gridDim.y >> slots) : slots) {
    MemT* vec = reinterpret_cast<MemT*>(logits + row * row_stride + sp.head);
    const int32_t* window = context + row * width;
    VecT buf[kU];
    if (first + kThreads * kU <= full) {
      // Whole tile inside the row: no per-vector guards, all loads in flight at once.
#pragma unroll
      for (int u = 0; u < kU; ++u) buf[u] = stream_load(vec + first + u * kThreads + threadIdx.x);
      const RowSeed<kW> rs = row_seed<kContext, kW>(key, window, width);
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const uint32_t j = first + u * kThreads + threadIdx.x;
        stream_store(vec + j, bias_vec_context(buf[u], j + jbase, rs.seed, tm1, delta));
      }
    } else {
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const uint32_t j = first + u * kThreads + threadIdx.x;
        if (j < full) buf[u] = stream_load(vec + j);
      }
      const RowSeed<kW> rs = row_seed<kContext, kW>(key, window, width);
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const uint32_t j = first + u * kThreads + threadIdx.x;
        if (j < full) stream_store(vec + j, bias_vec_context(buf[u], j + jbase, rs.seed, tm1, delta));
      }
    }
  }
}

// One token per lane, one row per y, either seeding, any start.  For launches that leave the
// chip mostly idle, where the time is that of a lane's chain of instructions: a vector's
// four or eight tokens lengthen it, and the workgroup column for the edges of a row that has
// some adds 0.3-0.5 us (16 x 4001 fp32, context: 2.25 us, 2.88 with vectors; 1 x 32000: 2.04,
// 2.23; self-salt width 4 2.29, 2.64).
template <typename T, int kSeeding, int kW>
__global__ void __launch_bounds__(kThreads)
watermark_token_kernel(T* __restrict__ logits, int64_t row_stride, uint32_t V,
                       int64_t B, const int32_t* __restrict__ context, int width, uint64_t key,
                       uint32_t tm1, float delta, uint32_t vbase) {
  const uint32_t v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= V) return;
  for (int64_t row = blockIdx.y; row < B; row += gridDim.y) {
    T* p = logits + row * row_stride + v;
    const T l = *p;
    const RowSeed<kW> rs = row_seed<kSeeding, kW>(key, context + row * width, width);
    *p = bias_elem(l, delta, is_green(draw<kSeeding>(rs, vbase + v), tm1));
  }
}

// ---------------------------------------------------------------------------
// Self-salt watermark.  The rows of a workgroup share their columns, so a candidate's J(v)
// and the row-independent term key*J(v)*J(v) of its seed are computed once per lane and
// reused for every row; the window terms key*J(p_i)*J(v), the minimum and the Philox draw
// are per row.
// ---------------------------------------------------------------------------
template <int kW>
__device__ __forceinline__ void quad_draws(uint32_t (&x)[4], uint32_t c, const CandTerm (&ct)[4],
                                           const RowSeed<kW>& rs) {
  x[0] = philox_block_lane<6>(c, key_of(self_salt_seed_t(rs, ct[0]))).w0;
  x[1] = philox_block_lane<6>(c, key_of(self_salt_seed_t(rs, ct[1]))).w1;
  x[2] = philox_block_lane<6>(c, key_of(self_salt_seed_t(rs, ct[2]))).w2;
  x[3] = philox_block_lane<6>(c, key_of(self_salt_seed_t(rs, ct[3]))).w3;
}
__device__ __forceinline__ f32x4 bias_quad(f32x4 l, const uint32_t (&x)[4], uint32_t tm1, float delta) {
  return f32x4{bias_f32(l.x, delta, is_green(x[0], tm1)), bias_f32(l.y, delta, is_green(x[1], tm1)),
               bias_f32(l.z, delta, is_green(x[2], tm1)), bias_f32(l.w, delta, is_green(x[3], tm1))};
}
__device__ __forceinline__ u32x2 bias_quad(u32x2 l, const uint32_t (&x)[4], uint32_t tm1, float delta) {
  return u32x2{bias_bf16x2(l.x, delta, is_green(x[0], tm1), is_green(x[1], tm1)),
               bias_bf16x2(l.y, delta, is_green(x[2], tm1), is_green(x[3], tm1))};
}

// Grid: x = tile of kThreads * kU quads of a row, y = a slot that takes the rows y, y + slots,
// ...; then grid rows for the edge columns.  The candidate terms depend on the columns only, so a workgroup
// computes them once, while its first row's loads are in flight, and uses them for every
// row it takes.  Bound by VALU issue: at width 4 a logit costs about 75 instructions, 51
// of them its Philox block.  The window is a template parameter, so the minimum is a
// straight chain that the compiler interleaves over a quad's four tokens (with a runtime
// width the chain branched and each compare waited out its hazard: 64 x 151936 fp32, width
// 4, 25.0 against 23.4 us).  bf16 takes 8-byte quads, not 16-byte vectors: half the terms
// per lane, 8 waves per SIMD instead of 4 (96.8 -> 77.9 us at 256 x 152064, width 4).
// Several rows at once per workgroup (their loads and draws side by side) measured slower
// than one after another at every size.
// Rows of whole quads have an instantiation of their own: beside the edges' code the main
// path runs slower, in as many registers (129 x 19648, width 4, us: bf16 9.36 with it, 9.12
// without; fp32 9.40, 9.26).
template <typename T, int kU, int kW, bool kEdges>
__global__ void __launch_bounds__(kThreads)
watermark_ss_rows_kernel(T* __restrict__ logits, int64_t row_stride, uint32_t V, int64_t B,
                         const int32_t* __restrict__ context, uint64_t key, uint32_t tm1, float delta,
                         uint32_t vbase, uint32_t slots) {
  using QuadT = typename QuadOf<T>::Value;
  using MemT = typename QuadOf<T>::Memory;
  const RowSplit sp = row_split<4>(V, vbase);
  const uint32_t full = sp.full;
  const uint32_t first = blockIdx.x * (kThreads * kU);
  const uint32_t id_first = first + sp.id;   // the tile's first quad counted in token ids
  const bool whole = first + kThreads * kU <= full;
  if (kEdges && blockIdx.y >= slots) {
    watermark_edges<T, kSelfSalt, kW, 4>(logits, row_stride, sp, B, context, kW, key, tm1, delta, vbase,
                                         blockIdx.y - slots, gridDim.y - slots);
    return;
  }
  CandTerm ct[kU][4];
  bool have_terms = false;
  for (int64_t row = blockIdx.y; row < B; row += slots) {
    MemT* quads = reinterpret_cast<MemT*>(logits + row * row_stride + sp.head);
    QuadT buf[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint32_t j = first + u * kThreads + threadIdx.x;
      if (whole || j < full) buf[u] = stream_load(quads + j);
    }
    if (!have_terms) {
      have_terms = true;
#pragma unroll
      for (int u = 0; u < kU; ++u)
#pragma unroll
        for (uint32_t e = 0; e < 4u; ++e)
          ct[u][e] = cand_term(key, (id_first + u * kThreads + threadIdx.x) * 4u + e);
    }
    const RowSeed<kW> rs = row_seed<kSelfSalt, kW>(key, context + row * kW, kW);
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint32_t j = first + u * kThreads + threadIdx.x;
      if (whole || j < full) {
        uint32_t x[4];
        quad_draws(x, id_first + u * kThreads + threadIdx.x, ct[u], rs);
        stream_store(quads + j, bias_quad(buf[u], x, tm1, delta));
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Self-salt watermark, fp32 or bf16, window of one token, by split terms over a slab
// of rows.  The seed of (row, v) is the smaller of the row term key*J(p)*J(v) and the
// self term key*J(v)*J(v) (Sec. 2.3 with the window {p, v}); the self term, and so
// the draw whenever it is the smaller one (about half of the pairs), is the same in
// every row.  A wave owns 64 16-byte vectors of a row (one per lane: 256 fp32 or 512
// bf16 columns) over a slab of up to kRows rows (12, or 8 or 6 for launches that
// taller slabs would leave with too few workgroups):
//  1. each lane draws its vector's self-term blocks (4 or 8) once and writes those
//     decisions into the slab's decision map (a byte per row and column, a lane's
//     columns in one word, or two for bf16) for every row;
//  2. one token position q of the vector at a time, the lanes whose row term is
//     smaller append (row term, map word, lane) to the wave's queue (ballot + mbcnt
//     give consecutive entries), and a queue holding 64 pairs is drained at once: 64
//     Philox draws side by side, each decision written over its map byte; the last
//     partial chunk is drained after the slab's last row;
//  3. each row's vector is biased from its map word and stored.
// The Philox counter and word are compile-time functions of q in every draw (q is a
// template argument), so each block keeps only the work its word needs.  Per logit this
// draws about 0.57 blocks instead of 1; the queueing costs about 9 instructions.
// ---------------------------------------------------------------------------
constexpr uint32_t kSlabQueue = 128;   // queue entries: fewer than 64 left + one row's 64
// Map words per row: one more than the lanes, so that the same lane's words in
// adjacent rows fall in different LDS banks.
constexpr uint32_t kSlabMapStride = 65;
constexpr int kSlabLoadRows = 4;       // rows whose logits are loaded together in step 3

// l + delta where bit `bit` of `bits` is set, l's own bits elsewhere: the bit widened
// to a full mask by a sign-extending field extract, then a bitwise select.
__device__ __forceinline__ float bias_bit(float l, float delta, uint32_t bits, int bit) {
  const uint32_t m = static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int>(bits), bit, 1));
  return __uint_as_float(
      __builtin_amdgcn_bitop3_b32(m, __float_as_uint(l + delta), __float_as_uint(l), 0xCA));
}

template <int kQ>
__device__ __forceinline__ uint32_t word_of(const Block& b) {
  return kQ == 0 ? b.w0 : kQ == 1 ? b.w1 : kQ == 2 ? b.w2 : b.w3;
}

// A queued pair: the row term (the Philox key, two words), its map word and the lane
// that queued it; one 16-byte record, one address and one LDS operation each way.
typedef uint32_t SlabEntry __attribute__((ext_vector_type(4)));

// One wave's LDS: the queue, the decision map (kPer bytes per row and lane: the
// decisions of a lane's kPer tokens), and each row's key * J(p).
template <int kRows, int kPer>
struct SlabLds {
  SlabEntry queue[kSlabQueue];
  uint32_t map[kRows * kSlabMapStride * (kPer / 4)];
  alignas(16) uint64_t kjp[kRows + 2];  // two spares for the read-ahead
};

// Draws the first n (<= 64) queue entries of token position kE (of the kPer tokens
// of a lane's vector), one per lane, writes each decision over its map byte, and
// moves entries 64 .. pending-1 to the front.  Lanes past n read entries inside the
// queue and store nothing.
template <int kE, int kRows, int kPer>
__device__ __forceinline__ void slab_drain(SlabLds<kRows, kPer>& s, uint32_t n, uint32_t pending,
                                           uint32_t lane, uint32_t jid0, uint32_t tm1) {
  const SlabEntry e = s.queue[lane];
  SlabEntry e2;  // read and written back only where `move` holds
  const bool move = lane + 64u < pending;
  if (move) e2 = s.queue[lane + 64u];
  // the pair's token is kPer * (jid0 + lane that queued it) + kE: Philox counter
  // (kPer / 4) * (jid0 + lane) + kE / 4, word kE mod 4
  const uint32_t x = word_of<kE % 4>(philox_block_lane<6>(
      (kPer / 4) * (jid0 + e.w) + static_cast<uint32_t>(kE / 4), Key{e.x, e.y}));
  if (lane < n)
    reinterpret_cast<uint8_t*>(s.map)[kPer * e.z + kE] = static_cast<uint8_t>(is_green(x, tm1));
  if (move) s.queue[lane] = e2;
}

// Queues the pairs of one row and token position kE whose row term kjp * J(v) is
// below `bound`, and drains the queue when it holds 64.
template <int kE, int kRows, int kPer>
__device__ __forceinline__ void slab_enqueue(SlabLds<kRows, kPer>& s, uint32_t& pending, uint64_t kjp,
                                             uint32_t jv, uint64_t bound, uint32_t map_word,
                                             uint32_t lane, uint32_t jid0, uint32_t tm1) {
  const uint64_t t = lane_mul_64x32(kjp, jv);
  // the lanes with t < bound, as one wave mask (the compiler shares the compare
  // with the branch below)
  const uint64_t mask = __builtin_amdgcn_uicmpl(t, bound, 36 /* unsigned less than */);
  if (t < bound) {
    const uint32_t at = pending + __builtin_amdgcn_mbcnt_hi(
                                      static_cast<uint32_t>(mask >> 32),
                                      __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
    s.queue[at] = SlabEntry{static_cast<uint32_t>(t), static_cast<uint32_t>(t >> 32), map_word, lane};
  }
  pending += static_cast<uint32_t>(__builtin_popcountll(mask));
  // LDS operations of one wave complete in order; the barriers only keep the
  // compiler from moving them across the passes.
  __builtin_amdgcn_wave_barrier();
  if (pending >= 64u) {
    slab_drain<kE, kRows, kPer>(s, 64u, pending, lane, jid0, tm1);
    pending -= 64u;
    __builtin_amdgcn_wave_barrier();
  }
}

// Token position kE over the rows of the slab: queue, drain at 64, drain the rest.
template <int kE, int kRows, int kPer>
__device__ __forceinline__ void slab_position(SlabLds<kRows, kPer>& s, int rows, uint32_t jv, uint64_t bound,
                                              uint32_t lane, uint32_t jid0, uint32_t tm1) {
  uint32_t pending = 0u;  // wave-uniform
  // four rows per iteration, their key * J(p) by two broadcast LDS reads of two rows
  // each, each pair read one pair ahead into the registers the pair before it has
  // just freed (entries past the last row are spares: read, never used)
  typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
  u64x2 a = *reinterpret_cast<const u64x2*>(&s.kjp[0]);
  int r = 0;
#pragma nounroll
  for (; r + 3 < rows; r += 4) {
    const u64x2 b = *reinterpret_cast<const u64x2*>(&s.kjp[r + 2]);
    const uint32_t w0 = static_cast<uint32_t>(r) * kSlabMapStride + lane;
    slab_enqueue<kE, kRows, kPer>(s, pending, a.x, jv, bound, w0, lane, jid0, tm1);
    slab_enqueue<kE, kRows, kPer>(s, pending, a.y, jv, bound, w0 + kSlabMapStride, lane, jid0, tm1);
    a = *reinterpret_cast<const u64x2*>(&s.kjp[r + 4]);
    slab_enqueue<kE, kRows, kPer>(s, pending, b.x, jv, bound, w0 + 2 * kSlabMapStride, lane, jid0, tm1);
    slab_enqueue<kE, kRows, kPer>(s, pending, b.y, jv, bound, w0 + 3 * kSlabMapStride, lane, jid0, tm1);
  }
  if (r + 1 < rows) {
    const uint32_t w0 = static_cast<uint32_t>(r) * kSlabMapStride + lane;
    slab_enqueue<kE, kRows, kPer>(s, pending, a.x, jv, bound, w0, lane, jid0, tm1);
    slab_enqueue<kE, kRows, kPer>(s, pending, a.y, jv, bound, w0 + kSlabMapStride, lane, jid0, tm1);
    r += 2;
    a = *reinterpret_cast<const u64x2*>(&s.kjp[r]);
  }
  if (r < rows)
    slab_enqueue<kE, kRows, kPer>(s, pending, a.x, jv, bound,
                                  static_cast<uint32_t>(r) * kSlabMapStride + lane, lane, jid0, tm1);
  if (pending != 0u) slab_drain<kE, kRows, kPer>(s, pending, pending, lane, jid0, tm1);
  __builtin_amdgcn_wave_barrier();
}

// The bias of a bf16 pair from its two map bytes (bits blo and bhi of the decision
// word d): one fp32 add each, one rounding, the non-green half's bits kept.
__device__ __forceinline__ uint32_t bias_pair_bits(uint32_t pair, float delta, uint32_t d, int blo,
                                                   int bhi) {
  const uint32_t mlo = static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int>(d), blo, 1));
  const uint32_t mhi = static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int>(d), bhi, 1));
  const uint32_t take = __builtin_amdgcn_bitop3_b32(0x0000FFFFu, mlo, mhi, 0xCA);
  const uint32_t biased = to_bf16x2(__uint_as_float(pair << 16) + delta,
                                    __uint_as_float(pair & 0xFFFF0000u) + delta);
  return __builtin_amdgcn_bitop3_b32(take, biased, pair, 0xCA);
}

// Step 3 of a row's vector: the bias from the row's kPer map bytes.
__device__ __forceinline__ f32x4 slab_bias(f32x4 o, float delta, const uint32_t (&d)[1]) {
  o.x = bias_bit(o.x, delta, d[0], 0);
  o.y = bias_bit(o.y, delta, d[0], 8);
  o.z = bias_bit(o.z, delta, d[0], 16);
  o.w = bias_bit(o.w, delta, d[0], 24);
  return o;
}
__device__ __forceinline__ u32x4 slab_bias(u32x4 o, float delta, const uint32_t (&d)[2]) {
  o.x = bias_pair_bits(o.x, delta, d[0], 0, 8);
  o.y = bias_pair_bits(o.y, delta, d[0], 16, 24);
  o.z = bias_pair_bits(o.z, delta, d[1], 0, 8);
  o.w = bias_pair_bits(o.w, delta, d[1], 16, 24);
  return o;
}

// The kPer token positions of a lane's vector, one after another.
template <int kE, int kRows, int kPer>
__device__ __forceinline__ void slab_positions(SlabLds<kRows, kPer>& s, int rows,
                                               const uint32_t (&jv)[kPer],
                                               const uint64_t (&bound)[kPer], uint32_t lane,
                                               uint32_t jid0, uint32_t tm1) {
  if constexpr (kE < kPer) {
    slab_position<kE, kRows, kPer>(s, rows, jv[kE], bound[kE], lane, jid0, tm1);
    slab_positions<kE + 1, kRows, kPer>(s, rows, jv, bound, lane, jid0, tm1);
  }
}

// Grid: x = tile of kThreads vectors (4 waves of 256 vectors), y = a slot taking the
// slabs y, y + slots, ... of kRows rows; then grid rows for the edge columns.  T: float (4 tokens a vector) or bf16
// bits (8).  Rows of whole vectors have an instantiation of their own (kEdges false): the
// path of the other columns in front of the tiles cost every wave its test and 0.8 %
// (256 x 152064 fp32: 64.9 us without it, 65.5 with; 1024: 237.1 / 238.7).
template <typename T, int kRows, bool kEdges>
__global__ void __launch_bounds__(kThreads)
watermark_ss_slab_kernel(T* __restrict__ logits, int64_t row_stride, uint32_t V, int64_t B,
                         const int32_t* __restrict__ context, uint64_t key, uint32_t tm1,
                         float delta, uint32_t vbase, uint32_t slots) {
  using VecT = typename VecOf<T>::Value;
  using MemT = typename VecOf<T>::Memory;
  constexpr int kPer = 16 / sizeof(T);  // tokens a vector
  constexpr int kWords = kPer / 4;      // map words (and Philox counters) a vector
  __shared__ SlabLds<kRows, kPer> lds[kThreads / 64];
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  SlabLds<kRows, kPer>& s = lds[wave];
  const RowSplit sp = kEdges ? row_split<kPer>(V, vbase) : RowSplit{0u, V / kPer, 0u, vbase / kPer};
  const uint32_t full = sp.full;
  if (kEdges && blockIdx.y >= slots) {
    watermark_edges<T, kSelfSalt, 1, kPer>(logits, row_stride, sp, B, context, 1, key, tm1, delta, vbase,
                                           blockIdx.y - slots, gridDim.y - slots);
    return;
  }
  const uint32_t j0 = blockIdx.x * kThreads + wave * 64u;  // the wave's first vector
  const uint32_t j = j0 + lane;
  const bool active = j < full;
  const uint32_t jid0 = j0 + sp.id;  // in token ids / kPer
  const uint32_t jid = jid0 + lane;
  // the lane's tokens: J(v), and the self term as the queueing bound (0, which no row
  // term is below, for a lane past the row's last whole vector)
  uint32_t jv[kPer];
  uint64_t bound[kPer];
  uint32_t self_word[kWords];
  {
    uint64_t self[kPer];
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      jv[e] = jenkins32(jid * kPer + static_cast<uint32_t>(e));
      self[e] = mul_64x64(key, wide_mul(jv[e], jv[e]));
      bound[e] = active ? self[e] : 0u;
    }
#pragma unroll
    for (int w = 0; w < kWords; ++w) {
      const uint32_t c = jid * kWords + static_cast<uint32_t>(w);  // Philox counter
      self_word[w] =
          static_cast<uint32_t>(is_green(word_of<0>(philox_block_lane<6>(c, key_of(self[4 * w]))), tm1)) |
          static_cast<uint32_t>(is_green(word_of<1>(philox_block_lane<6>(c, key_of(self[4 * w + 1]))), tm1)) << 8 |
          static_cast<uint32_t>(is_green(word_of<2>(philox_block_lane<6>(c, key_of(self[4 * w + 2]))), tm1)) << 16 |
          static_cast<uint32_t>(is_green(word_of<3>(philox_block_lane<6>(c, key_of(self[4 * w + 3]))), tm1)) << 24;
    }
  }
  T* first_vec = logits + sp.head;
  const int64_t slabs = (B + kRows - 1) / kRows;
  for (int64_t g = blockIdx.y; g < slabs; g += slots) {
    const int64_t row0 = g * kRows;
    const int rows = static_cast<int>(B - row0 < kRows ? B - row0 : kRows);
    // step 1: the self decisions for every row, and each row's key * J(p)
#pragma nounroll
    for (int r = 0; r < rows; ++r) {
#pragma unroll
      for (int w = 0; w < kWords; ++w)
        s.map[(static_cast<uint32_t>(r) * kSlabMapStride + lane) * kWords + w] = self_word[w];
    }
    if (lane < static_cast<uint32_t>(rows))
      s.kjp[lane] = key * static_cast<uint64_t>(jenkins32(static_cast<uint32_t>(context[row0 + lane])));
    __builtin_amdgcn_wave_barrier();
    // step 2: the pairs whose row term is smaller, one token position at a time
    slab_positions<0, kRows, kPer>(s, rows, jv, bound, lane, jid0, tm1);
    // step 3: bias and store, kSlabLoadRows rows' loads in flight at a time
    if (active) {
      for (int r0 = 0; r0 < rows; r0 += kSlabLoadRows) {
        VecT buf[kSlabLoadRows];
        uint32_t dec[kSlabLoadRows][kWords];
#pragma unroll
        for (int k = 0; k < kSlabLoadRows; ++k) {
          if (r0 + k < rows) {
            buf[k] = stream_load(reinterpret_cast<const MemT*>(first_vec + (row0 + r0 + k) * row_stride) + j);
#pragma unroll
            for (int w = 0; w < kWords; ++w)
              dec[k][w] = s.map[(static_cast<uint32_t>(r0 + k) * kSlabMapStride + lane) * kWords + w];
          }
        }
#pragma unroll
        for (int k = 0; k < kSlabLoadRows; ++k) {
          if (r0 + k < rows)
            stream_store(reinterpret_cast<MemT*>(first_vec + (row0 + r0 + k) * row_stride) + j,
                         slab_bias(buf[k], delta, dec[k]));
        }
      }
    }
    __builtin_amdgcn_wave_barrier();  // the next slab rewrites the map
  }
}

// ---------------------------------------------------------------------------
// Greedy decoding fused with the watermark: the argmax of each watermarked row in
// one read-only pass.  A row is cut into segments; one workgroup scans a segment,
// keeps a running (value, index) per lane, reduces them and writes one partial
// (value bits, index) to the workspace.  A read-out kernel then reduces the
// partials of each row.  Candidates compare through a 64-bit key: the high word
// orders the values (every NaN above +inf, -0 equal to +0), the low word is
// ~index, so the maximum key is the largest value at its smallest index.
// ---------------------------------------------------------------------------
// 16-byte vectors per lane in a workgroup segment of the fused decoding pass, and the
// sub-batches that a segment is taken in.  A longer segment gives each wave a larger sample
// for its bounds, but every lane holds a sub-batch in registers.  Sampling fp32, 256 x
// 152064: 4 / 6 / 8 / 12 vectors 44.4 / 37.7 / 38.2 / 40.7 us; sampling bf16, 160 x 152064:
// 4 / 5 / 6 / 8 vectors 26.0 / 25.4 / 25.5 / 27.9 us; greedy fp32, 256 x 152064: 28.0 us from
// 4 to 8.  Greedy bf16 takes two sub-batches, the second's loads in flight while the first
// is scored: 900 x 152064, one / two 52.2 / 50.3 us (60.3 before).
#ifndef SBW_DECODE_VECS_F32_GREEDY
#define SBW_DECODE_VECS_F32_GREEDY 6
#endif
#ifndef SBW_DECODE_VECS_F32
#define SBW_DECODE_VECS_F32 8          // sampling
#endif
#ifndef SBW_DECODE_VECS_BF16
#define SBW_DECODE_VECS_BF16 4         // greedy
#endif
#ifndef SBW_DECODE_VECS_BF16_SAMPLE
#define SBW_DECODE_VECS_BF16_SAMPLE 5
#endif
#ifndef SBW_DECODE_SUBS_BF16
#define SBW_DECODE_SUBS_BF16 2         // greedy; the others take one
#endif
// Greedy fp32 decoding of more than the Infinity Cache holds: unused LDS that leaves a CU 6
// workgroups instead of 8.  With all 8 streaming, the reads crowd each other out (900 x
// 152064: 8 / 7 / 6 / 5 of them 84.6 / 83.7 / 82.0 / 84.8 us; 256 x 152064, 27.6 / 27.4 /
// 27.9 / 29.3; bf16 is fastest with all).
constexpr uint32_t kCrowdedLds = 16000;
constexpr int64_t kArgmaxSegElems = kThreads * 8;   // the shortest segment the workspace holds

__device__ __forceinline__ uint32_t order_bits(float f) {
  uint32_t b = __float_as_uint(f);
  if (f != f) return 0xFFFFFFFFu;
  if (b == 0x80000000u) b = 0u;
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ __forceinline__ uint64_t arg_key(float f, uint32_t v) {
  return (static_cast<uint64_t>(order_bits(f)) << 32) | static_cast<uint32_t>(~v);
}

// Running argmax of one lane.  `any` is false until the lane has seen an element.
struct LaneBest {
  float v;
  uint32_t i;
  bool any;
};

__device__ __forceinline__ LaneBest lane_best_init() { return LaneBest{0.0f, 0u, false}; }

// The lane sees its indices in any order: a larger value wins, any NaN wins over numbers,
// equal values (-0 == +0) and NaNs go to the smaller index.
__device__ __forceinline__ void consider_any_order(LaneBest& b, float x, uint32_t i) {
  const int xn = static_cast<int>(x != x), bn = static_cast<int>(b.v != b.v);
  const int first = static_cast<int>(i < b.i);
  const bool take = static_cast<bool>(static_cast<int>(!b.any) | static_cast<int>(x > b.v) |
                                      (static_cast<int>(x == b.v) & first) |
                                      (xn & ((1 - bn) | first)));
  b.v = take ? x : b.v;
  b.i = take ? i : b.i;
  b.any = true;
}

__device__ __forceinline__ float widen(float x) { return x; }
__device__ __forceinline__ float widen(uint16_t x) { return __uint_as_float(static_cast<uint32_t>(x) << 16); }

// A partial result: value bits in the high word, index in the low word (0 = none is
// never produced: a workgroup's segment always holds at least one element).
__device__ __forceinline__ uint64_t pack_partial(float v, uint32_t i) {
  return (static_cast<uint64_t>(__float_as_uint(v)) << 32) | i;
}
__device__ __forceinline__ uint64_t partial_key(uint64_t p) {
  return arg_key(__uint_as_float(static_cast<uint32_t>(p >> 32)), static_cast<uint32_t>(p));
}

// Wave-wide maximum of 64-bit keys with their 64-bit payloads, by DPP moves (quad
// permutes, row mirrors, then row broadcasts that carry the maximum to lane 63); no
// index arithmetic or LDS round trips.  Lanes a move does not reach see key 0, which
// never wins.  The result is read from lane 63 into every lane.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ void dpp_argmax_step(uint64_t& k, uint64_t& p) {
  const uint32_t k0 = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
      0, static_cast<int>(static_cast<uint32_t>(k)), kCtrl, kRowMask, 0xF, false));
  const uint32_t k1 = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
      0, static_cast<int>(static_cast<uint32_t>(k >> 32)), kCtrl, kRowMask, 0xF, false));
  const uint32_t p0 = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
      0, static_cast<int>(static_cast<uint32_t>(p)), kCtrl, kRowMask, 0xF, false));
  const uint32_t p1 = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
      0, static_cast<int>(static_cast<uint32_t>(p >> 32)), kCtrl, kRowMask, 0xF, false));
  const uint64_t ok = (static_cast<uint64_t>(k1) << 32) | k0;
  if (ok > k) {
    k = ok;
    p = (static_cast<uint64_t>(p1) << 32) | p0;
  }
}
__device__ __forceinline__ uint64_t readlane63(uint64_t x) {
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(x)), 63));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(x >> 32)), 63));
  return (static_cast<uint64_t>(hi) << 32) | lo;
}
__device__ __forceinline__ void wave_argmax(uint64_t& k, uint64_t& p) {
  dpp_argmax_step<0xB1, 0xF>(k, p);    // quad_perm [1,0,3,2]
  dpp_argmax_step<0x4E, 0xF>(k, p);    // quad_perm [2,3,0,1]
  dpp_argmax_step<0x141, 0xF>(k, p);   // row_half_mirror
  dpp_argmax_step<0x140, 0xF>(k, p);   // row_mirror
  dpp_argmax_step<0x142, 0xA>(k, p);   // row_bcast:15 into rows 1 and 3
  dpp_argmax_step<0x143, 0xC>(k, p);   // row_bcast:31 into rows 2 and 3
  k = readlane63(k);
  p = readlane63(p);
}

// Block-wide argmax of the lanes' running bests; thread 0 stores the partial.
__device__ __forceinline__ void block_argmax_store(const LaneBest& lb, uint64_t* out,
                                                   uint64_t* lds_key, uint64_t* lds_part) {
  uint64_t k = 0u, p = 0u;
  if (__any(lb.any)) {   // most often the queue's tokens all went to the first wave
    k = lb.any ? arg_key(lb.v, lb.i) : 0u;
    p = pack_partial(lb.v, lb.i);
    wave_argmax(k, p);
  }
  if (threadIdx.x % 64 == 0) {
    lds_key[threadIdx.x / 64] = k;
    lds_part[threadIdx.x / 64] = p;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t bk = lds_key[0], bp = lds_part[0];
#pragma unroll
    for (int w = 1; w < kThreads / 64; ++w)
      if (lds_key[w] > bk) { bk = lds_key[w]; bp = lds_part[w]; }
    *out = bp;
  }
  __syncthreads();  // the LDS slots are reused by the next row of this workgroup
}

// Skipping elements that cannot win.  An element's watermarked value is either its
// logit x or bias(x) (the value it takes when green), and bias is non-decreasing in
// x for both dtypes (one rounded add; bf16 rounding is monotone too).  So if m is
// the largest logit of some set of elements, one of them ends at least at
// lb = min(m, bias(m)), and an element with x < lb and bias(x) < lb can be neither
// the maximum nor tied with it: its colour need not be drawn.  A NaN compares false
// and is always kept (it wins), so NaN logits never make the test skip anything;
// delta is finite, so bias(x) is NaN only when x is.
// The lower bound from the largest logit m (-inf when there is none).
__device__ __forceinline__ float reach_bound(float m, float delta, float) {
  return fminf(m, m + delta);
}
__device__ __forceinline__ float reach_bound(float m, float delta, uint16_t) {
  const uint32_t b = __float_as_uint(m) >> 16;   // m is a widened bf16
  return fminf(m, widen(bias_bf16(static_cast<uint16_t>(b), delta, true)));
}

// A logit below which neither candidate value reaches lb (never a NaN): x + dplus, rounded
// (to 24 or 8 significant bits), is at most x + dplus + rel * (|lb| + dplus) where it reaches
// lb.  A bound of +inf is taken as the largest finite float, which a token that reaches it
// reaches too; sums that overflow here give -inf, which keeps every token.
__device__ __forceinline__ float reach_threshold(float lb, float dplus, float) {
  const float c = fminf(lb, FLT_MAX);
  return (c - dplus) - (0x1p-21f * fabsf(c) + 0x1p-21f * dplus);
}
__device__ __forceinline__ float reach_threshold(float lb, float dplus, uint16_t) {
  const float c = fminf(lb, FLT_MAX);
  return (c - dplus) - (0x1p-7f * fabsf(c) + 0x1p-7f * dplus) - 0x1p-130f;
}
// Sampling: what a token's bound without kNoiseBitsOffset has to reach for a score of at
// least lb (the roundings of the bound are far below the relative term).
__device__ __forceinline__ float reach_noise_threshold(float lb) {
  const float c = fminf(lb, FLT_MAX);
  return (c - kNoiseBitsOffset) - 0x1p-20f * (fabsf(c) + 256.0f);
}

// What a pass maximises: the watermarked logit (greedy decoding), or, for sampling,
// that logit times 1/T plus the token's Gumbel noise (the Gumbel-max trick).
template <bool kSample>
struct Score {
  uint64_t seed;    // sampling: the row's noise seed
  float inv_t;      // sampling: 1 / temperature
};

// A token's larger candidate logit, max(x, bias(x)): bias(x) for a positive delta, else x;
// either way x + dplus rounded to the logits' type, dplus = max(delta, 0) (x + 0 only turns
// -0 into +0).  Non-decreasing in x.
__device__ __forceinline__ float upper_logit(float x, float dplus, float) { return x + dplus; }
__device__ __forceinline__ float upper_logit(float x, float dplus, uint16_t) {   // x: a widened bf16
  return __uint_as_float(to_bf16x2(x + dplus, 0.0f) << 16);
}
__device__ __forceinline__ void upper_logits(f32x4 o, float dplus, float (&phi)[4]) {
  phi[0] = o.x + dplus;
  phi[1] = o.y + dplus;
  phi[2] = o.z + dplus;
  phi[3] = o.w + dplus;
}
__device__ __forceinline__ void upper_logits(u32x4 o, float dplus, float (&phi)[8]) {
  const uint32_t w[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t g = to_bf16x2(__uint_as_float(w[q] << 16) + dplus,
                                 __uint_as_float(w[q] & 0xFFFF0000u) + dplus);
    phi[2 * q] = __uint_as_float(g << 16);
    phi[2 * q + 1] = __uint_as_float(g & 0xFFFF0000u);
  }
}

// Largest of a vector's values, NaN when one of them is.
__device__ __forceinline__ float max3_nan(float a, float b, float c) {
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}
__device__ __forceinline__ float vec_max(const float (&x)[4]) {
  return __builtin_elementwise_maximum(max3_nan(x[0], x[1], x[2]), x[3]);
}
__device__ __forceinline__ float vec_max(const float (&x)[8]) {
  return __builtin_elementwise_maximum(max3_nan(max3_nan(max3_nan(x[0], x[1], x[2]), x[3], x[4]), x[5], x[6]), x[7]);
}
__device__ __forceinline__ float vec_max(f32x4 o) {
  const float x[4] = {o.x, o.y, o.z, o.w};
  return vec_max(x);
}
__device__ __forceinline__ float vec_max(u32x4 o) {
  const uint32_t w[4] = {o.x, o.y, o.z, o.w};
  float x[8];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    x[2 * q] = __uint_as_float(w[q] << 16);
    x[2 * q + 1] = __uint_as_float(w[q] & 0xFFFF0000u);
  }
  return vec_max(x);
}

// The larger of a and b; a NaN loses.  v_max_f32 on the raw values: the compiler's fmaxf
// would first canonicalise every loaded value.  A signalling NaN may make the result NaN,
// which only turns the skip tests built on it off.
__device__ __forceinline__ float max_raw(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// Largest value over the wave, by DPP moves on order-preserving integer keys (no
// index arithmetic or LDS round trips): within quads, half rows and rows, then row
// broadcasts carry the maximum to lane 63.  A NaN lane may make the result NaN,
// which makes every bound test above keep its token.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ int dpp_max_step(int k) {
  return max(k, __builtin_amdgcn_update_dpp(static_cast<int>(0x80000000u), k, kCtrl, kRowMask, 0xF, false));
}
__device__ __forceinline__ float wave_max(float v) {
  int k = __float_as_int(v);
  k ^= (k >> 31) & 0x7FFFFFFF;
  k = dpp_max_step<0xB1, 0xF>(k);    // quad_perm [1,0,3,2]
  k = dpp_max_step<0x4E, 0xF>(k);    // quad_perm [2,3,0,1]
  k = dpp_max_step<0x141, 0xF>(k);   // row_half_mirror
  k = dpp_max_step<0x140, 0xF>(k);   // row_mirror
  k = dpp_max_step<0x142, 0xA>(k);   // row_bcast:15 into rows 1 and 3
  k = dpp_max_step<0x143, 0xC>(k);   // row_bcast:31 into rows 2 and 3
  k = __builtin_amdgcn_readlane(k, 63);
  return __int_as_float(k ^ ((k >> 31) & 0x7FFFFFFF));
}

__device__ __forceinline__ uint32_t raw_bits(float x) { return __float_as_uint(x); }
__device__ __forceinline__ uint32_t raw_bits(uint16_t x) { return x; }

// A vector of -inf, for the lanes past a row's last vector.
__device__ __forceinline__ f32x4 lowest_vec(f32x4) { return f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY}; }
__device__ __forceinline__ u32x4 lowest_vec(u32x4) { return u32x4{0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u}; }

// Element e of a vector, widened.
__device__ __forceinline__ float elem(f32x4 o, int e) {
  const float w[4] = {o.x, o.y, o.z, o.w};
  return w[e];
}
__device__ __forceinline__ float elem(u32x4 o, int e) {
  const uint32_t w[4] = {o.x, o.y, o.z, o.w};
  return __uint_as_float((e & 1) ? (w[e >> 1] & 0xFFFF0000u) : (w[e >> 1] << 16));
}

// The raw bits of element e of a vector (fp32 bits, or bf16 bits in the low half).
__device__ __forceinline__ uint32_t raw_elem(f32x4 o, int e) {
  const float w[4] = {o.x, o.y, o.z, o.w};
  return __float_as_uint(w[e]);
}
__device__ __forceinline__ uint32_t raw_elem(u32x4 o, int e) {
  const uint32_t w[4] = {o.x, o.y, o.z, o.w};
  return (e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xFFFFu);
}
__device__ __forceinline__ float from_raw(uint32_t r, float) { return __uint_as_float(r); }
__device__ __forceinline__ uint16_t from_raw(uint32_t r, uint16_t) { return static_cast<uint16_t>(r); }

// The noise draws of vector j: 4 tokens (fp32) or 8 (bf16), one block per 4 tokens
// as CBRNG lays them out.
__device__ __forceinline__ void noise_words(uint32_t j, const RoundKeys& k, uint32_t (&x)[4]) {
  const Block n = philox_block(j, k);
  x[0] = n.w0; x[1] = n.w1; x[2] = n.w2; x[3] = n.w3;
}
__device__ __forceinline__ void noise_words(uint32_t j, const RoundKeys& k, uint32_t (&x)[8]) {
  const Block n0 = philox_block(2u * j, k);
  const Block n1 = philox_block(2u * j + 1u, k);
  x[0] = n0.w0; x[1] = n0.w1; x[2] = n0.w2; x[3] = n0.w3;
  x[4] = n1.w0; x[5] = n1.w1; x[6] = n1.w2; x[7] = n1.w3;
}

// Appends a lane's token to the wave's queue at its rank among the lanes in mask.
__device__ __forceinline__ void enqueue(uint32_t* q_v, uint32_t* q_raw, uint32_t queued, uint64_t mask,
                                        uint32_t v, uint32_t raw) {
  const uint32_t pos = queued + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                                          __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
  q_v[pos] = v;
  q_raw[pos] = raw;
}

// The exact score of one queued token: colour, bias, noise.
template <typename T, int kSeeding, int kW, bool kSample>
__device__ __forceinline__ void score_entry(LaneBest& b, uint32_t v, uint32_t raw_bits,
                                            const RowSeed<kW>& rs, uint32_t tm1, int none_green,
                                            float delta, const Score<kSample>& sc) {
  const T raw = from_raw(raw_bits, T{});
  uint32_t x;
  if constexpr (kSeeding == kContext)
    x = block_word(philox_block(v >> 2, opaque_key(key_of(rs.seed))), v & 3u);
  else
    x = draw<kSelfSalt>(rs, v);
  const bool g = !none_green && is_green(x, tm1);
  const float l = widen(bias_elem(raw, delta, g));
  if constexpr (kSample) {
    const float noise = gumbel_of(block_word(philox_block(v >> 2, opaque_key(key_of(sc.seed))), v & 3u));
    consider_any_order(b, l * sc.inv_t + noise, v);
  } else {
    consider_any_order(b, l, v);
  }
}

// Scores the queued tokens of a wave, 64 at a time, one per lane.
template <typename T, int kSeeding, int kW, bool kSample>
__device__ __forceinline__ void score_queue(LaneBest& b, const uint32_t* q_v, const uint32_t* q_raw,
                                            uint32_t queued, const RowSeed<kW>& rs, uint32_t tm1,
                                            int none_green, float delta, const Score<kSample>& sc) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  for (uint32_t i = threadIdx.x % 64u; i < queued; i += 64u)
    score_entry<T, kSeeding, kW, kSample>(b, q_v[i], q_raw[i], rs, tm1, none_green, delta, sc);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Fused decoding: greedy (kSample false) or Gumbel-max sampling.  A segment is kSub
// sub-batches of kThreads * kN vectors, vector n of lane t at offset n * kThreads + t; a
// sub-batch is loaded while the one before it is scored.  The colour draw (and, sampling,
// the exact noise with its two logarithms) matters only for the few tokens that may still
// reach the wave's best score.  Per sub-batch:
//  1. greedy: with m the wave's largest logit, some token ends at least at
//     lb = min(m, bias(m)), and a token below reach_threshold(lb) stays under it;
//     sampling: lb from m with the noise's overall minimum, and a vector none of whose
//     tokens reaches lb even with the noise's overall maximum draws no noise (tested on
//     its largest logit); the others draw their noise, each token's score is bounded from
//     above by the bounds of its noise (noise_bits) and of its logit, and lb rises to
//     the wave's largest lower bound;
//  2. a vector whose largest bound reaches lb in some lane has its tokens tested one by
//     one, and those that reach lb join the wave's queue in LDS; a queue that would
//     overflow is scored exactly, one token per lane, and lb rises to the best of these
//     scores; at the end the four waves' queues are scored together.
// lb only rises.  A token left out scores below lb, which some token of the wave's
// share attains, so the partial equals that of a full scan.  Lanes see tokens out of index
// order, so their running argmax breaks ties by index.  Rows start anywhere, as in the
// watermark.
//
// Sampling is bound by VALU issue: 38 instructions for the noise block of 4 tokens and about
// 10 a token to bound it.  Testing vectors before tokens, the noise bound from the float's
// bits (4 instructions, a gap of 0.17 instead of 0.84 between its bounds, so fewer tokens
// queue) and the queue's count and the round keys in scalar registers took 256 x 152064
// fp32 from 42.9 to 38.5 us (1100 -> 870 VALU instructions a wave), bf16 160 x 152064 from
// 28.9 to 25.3.  Greedy reads at the memory's rate in large launches (bf16 900 x 152064:
// 60.3 -> 50.3 us, 5.4 TB/s).  Rows off 16 bytes took an element-wise kernel before that
// drew every token's colour: 48 x 128259, greedy bf16 self-salt width 4 / sampled fp32
// context, 27.5 -> 7.9 us, 31.3 -> 12.8 us.
//
// A delta that is large against the logits' spread puts most tokens within reach of step
// 1's bound; the exact scores then raise it past all but the green ones near the top
// (64 x 128256 N(0,2), delta 8, with that rise / without: greedy fp32 13.7 / 32.3 us, bf16
// 14.1 / 29.5; sampling fp32 19.6 / 48.2, bf16 31.3 / 45.7).
template <typename T, int kSeeding, int kN, int kSub, int kW, bool kSample>
__global__ void __launch_bounds__(kThreads)
decode_vec_kernel(const T* __restrict__ logits, int64_t row_stride, uint32_t V, int64_t B,
                  const int32_t* __restrict__ context, int width, uint64_t key, uint32_t tm1,
                  int none_green, float delta, const uint64_t* __restrict__ seeds, float inv_t,
                  uint32_t segments, uint64_t* __restrict__ partials, uint32_t vbase) {
  using VecT = typename VecOf<T>::Value;
  using MemT = typename VecOf<T>::Memory;
  constexpr int kE = 16 / sizeof(T);                 // tokens per vector
  const RowSplit sp = row_split<kE>(V, vbase);
  const uint32_t jbase = sp.id;                      // the first vector's token id / kE
  __shared__ uint64_t lds_key[kThreads / 64], lds_part[kThreads / 64];
  // Per wave: token ids, then raw logits.  The queue is scored whenever it holds more
  // than 64 tokens before a vector is queued, so it never holds more than 64 plus one
  // vector's worth (kE tokens in each of 64 lanes).
  constexpr uint32_t kQueueCap = 64u + 64u * kE;
  __shared__ uint32_t lds_queue[(kThreads / 64) * 2 * kQueueCap];
  __shared__ uint32_t lds_count[kThreads / 64];
  uint32_t* q_v = lds_queue + (threadIdx.x / 64u) * 2u * kQueueCap;
  uint32_t* q_raw = q_v + kQueueCap;
  constexpr uint32_t kSubVecs = kThreads * kN;       // vectors per sub-batch
  const uint32_t full = sp.full;
  const uint32_t segment = blockIdx.x;
  const uint32_t seg_base = segment * (kSubVecs * kSub);
  for (int64_t row = blockIdx.y; row < B; row += gridDim.y) {
    const T* row_ptr = logits + row * row_stride;
    const MemT* vec = reinterpret_cast<const MemT*>(row_ptr + sp.head);
    Score<kSample> sc{0u, inv_t};
    RoundKeys nk{};
    if constexpr (kSample) {
      sc.seed = seeds[row];
      nk = scalar_round_keys(key_of(sc.seed));
    }
    const RowSeed<kW> rs = row_seed<kSeeding, kW>(key, context + row * width, width);
    const float dt = fabsf(delta) * inv_t;
    const float dplus = delta > 0.0f ? delta : 0.0f;
    LaneBest best = lane_best_init();
    float lb = -INFINITY;           // the best score is at least lb (the same in every lane)
    uint32_t queued = 0;            // tokens in the wave's queue (the same in every lane)
    // The columns outside whole vectors (at most 14) are queued by the first wave of the
    // last segment, which has the fewest vectors and is never empty.  (Scored on their own
    // they cost 4 VGPRs a lane and with them a wave per SIMD: sampling 256 x 152064 fp32
    // 43.9 -> 50.2 us.)
    if (sp.edges() != 0u && segment + 1u == segments &&
        __builtin_amdgcn_readfirstlane(threadIdx.x / 64u) == 0u) {
      if (threadIdx.x < sp.edges()) {
        const uint32_t c = sp.template edge<kE>(threadIdx.x);   // column; the token id is vbase + c
        q_v[threadIdx.x] = vbase + c;
        q_raw[threadIdx.x] = raw_bits(row_ptr[c]);
      }
      queued = sp.edges();
    }
    // Sub-batch `sub` into registers; the next one is loaded while this one is scored.
    auto load_sub = [&](VecT (&buf)[kN], int sub) {
      // Opaque to the optimiser, so that no Philox work is hoisted out of the loops.
      uint32_t sub_first = seg_base + static_cast<uint32_t>(sub) * kSubVecs;
      asm volatile("" : "+s"(sub_first));
      if (sub_first + kSubVecs <= full) {
#pragma unroll
        for (int n = 0; n < kN; ++n) buf[n] = stream_load(vec + sub_first + n * kThreads + threadIdx.x);
      } else {
#pragma unroll
        for (int n = 0; n < kN; ++n) {
          const uint32_t j = sub_first + n * kThreads + threadIdx.x;
          buf[n] = lowest_vec(VecT{});
          if (j < full) buf[n] = stream_load(vec + j);
        }
      }
    };
    auto process_sub = [&](const VecT (&buf)[kN], int sub) {
      uint32_t sub_first = seg_base + static_cast<uint32_t>(sub) * kSubVecs;
      asm volatile("" : "+s"(sub_first));
      // The same sub-batch counted in token-id vectors (the row's first id is vbase).
      uint32_t id_first = sub_first + jbase;
      asm volatile("" : "+s"(id_first));
      const bool whole = sub_first + kSubVecs <= full;
      float m = -INFINITY;
      float vm[kN];                   // each vector's largest logit, NaN when it has one
#pragma unroll
      for (int n = 0; n < kN; ++n) {
        vm[n] = vec_max(buf[n]);
        m = max_raw(m, vm[n]);
      }
      float hi[kSample ? kN : 1][kE]; // sampling: the tokens' upper bounds, noise_bits apart
      float reach;                    // what a token's bound has to reach (the same in every lane)
      if constexpr (!kSample) {
        lb = fmaxf(lb, reach_bound(wave_max(m), delta, T{}));
        reach = reach_threshold(lb, dplus, T{});
      } else {
        const float lb0 = fmaxf(lb, reach_bound(wave_max(m), delta, T{}) * inv_t + kGumbelLo);
        float top = -INFINITY;        // the lane's largest hi
#pragma unroll
        for (int n = 0; n < kN; ++n) {
          const float most = upper_logit(vm[n], dplus, T{}) * inv_t + kGumbelHi;
          vm[n] = -INFINITY;          // from here on the vector's largest hi
#pragma unroll
          for (int e = 0; e < kE; ++e) asm("" : "=v"(hi[n][e]));   // any value: vm decides
          if (!(most < lb0)) {
            const uint32_t j = id_first + n * kThreads + threadIdx.x;
            uint32_t nw[kE];
            noise_words(j, nk, nw);
            upper_logits(buf[n], dplus, hi[n]);
#pragma unroll
            for (int e = 0; e < kE; ++e)
              hi[n][e] = __builtin_fmaf(noise_bits(nw[e]), -kNoiseBitsScale, hi[n][e] * inv_t);
            vm[n] = vec_max(hi[n]);
            top = max_raw(top, vm[n]);
          }
        }
        // The lane's token with the largest bound `up`, if its noise lies in the upper
        // range (as it must when `up` exceeds every logit of the lane by more than the
        // noise bound outside that range), scores at least up - gap - d: its noise is that
        // close to its bound, and its two candidate logits times 1/T differ by at most
        // |delta|/T plus roundings (of the bias, to 8 significant bits for bf16, of the
        // products and of these sums), which the relative term covers.  An infinite
        // `up` gives no bound.
        constexpr float kRel = sizeof(T) == 4 ? 0x1p-18f : 0x1p-7f;
        const float up = top + kNoiseBitsOffset;
        const float pm = upper_logit(m, dplus, T{}) * inv_t;
        const float slack = kNoiseGap + dt + kRel * (fabsf(up) + 18.0f + dt);
        const bool upper_range = up - pm > kNoiseUpperRange + 0x1p-18f * (fabsf(pm) + 18.0f);
        const float lb_lane = up < INFINITY && upper_range ? up - slack : -INFINITY;
        lb = fmaxf(lb0, wave_max(lb_lane));
        reach = reach_noise_threshold(lb);
      }

      // Queue the tokens whose upper bound reaches lb.  The counters are the same in
      // every lane.
#pragma unroll
      for (int n = 0; n < kN; ++n) {
        const uint32_t j = sub_first + n * kThreads + threadIdx.x;
        if (queued > 64u) {
          score_queue<T, kSeeding, kW, kSample>(best, q_v, q_raw, queued, rs, tm1, none_green, delta, sc);
          queued = 0;
          // the exact scores raise the bound (a NaN among them leaves it)
          lb = fmaxf(lb, wave_max(best.any ? best.v : -INFINITY));
          reach = kSample ? reach_noise_threshold(lb) : reach_threshold(lb, dplus, T{});
        }
        uint64_t lanes = __ballot(!(vm[n] < reach));
        if (!whole) lanes &= __ballot(j < full);
        if (lanes == 0u) continue;
        const uint32_t jid = id_first + n * kThreads + threadIdx.x;
#pragma unroll
        for (int e = 0; e < kE; ++e) {
          const uint64_t mask = __ballot(!((kSample ? hi[n][e] : elem(buf[n], e)) < reach)) & lanes;
          if (__builtin_amdgcn_inverse_ballot_w64(mask))
            enqueue(q_v, q_raw, queued, mask, jid * kE + e, raw_elem(buf[n], e));
          queued += static_cast<uint32_t>(__popcll(mask));
        }
      }
    };
    VecT buf0[kN], buf1[kN];
    load_sub(buf0, 0);
    for (int sub = 0; sub < kSub; sub += 2) {
      if (sub + 1 < kSub) load_sub(buf1, sub + 1);
      process_sub(buf0, sub);
      if (sub + 1 < kSub) {
        if (sub + 2 < kSub) load_sub(buf0, sub + 2);
        process_sub(buf1, sub + 1);
      }
    }
    // What is left in the four queues is scored together: entry i of their
    // concatenation goes to lane i % 64 of wave (i / 64) % 4, so a workgroup's few
    // candidates take one wave's pass instead of four.
    {
      const uint32_t lane = threadIdx.x % 64u, wave = threadIdx.x / 64u;
      if (lane == 0u) lds_count[wave] = queued;
      __syncthreads();
      uint32_t start[kThreads / 64 + 1];
      start[0] = 0u;
#pragma unroll
      for (int w = 0; w < kThreads / 64; ++w) start[w + 1] = start[w] + lds_count[w];
      const uint32_t total = start[kThreads / 64];
      for (uint32_t i = wave * 64u + lane; i < total; i += kThreads) {
        uint32_t w = 0;
#pragma unroll
        for (int k = 1; k < kThreads / 64; ++k) w += static_cast<uint32_t>(i >= start[k]);
        const uint32_t* wq = lds_queue + w * 2u * kQueueCap;
        const uint32_t off = i - start[w];
        score_entry<T, kSeeding, kW, kSample>(best, wq[off], wq[kQueueCap + off], rs, tm1, none_green,
                                               delta, sc);
      }
    }
    block_argmax_store(best, partials + row * segments + segment, lds_key, lds_part);
  }
}

// Decoding of short rows, which need no partials: kRowWaves waves score every token of a row,
// at most kShortSteps a lane, and store the winner, in one launch.  Bound by a lane's chain
// (window, colour, sampling two logarithms) in small launches, by VALU issue in large ones; the
// segment pass spends its fixed part (bounds, queues, a read-out launch) on few tokens.  us,
// segments / this: greedy fp32 1 x 37 4.5 / 2.2, 1000 x 513 6.6 / 4.1; sampling 5000 x 100 31.1 /
// 5.4, 1000 x 1001 8.5 / 7.3.
constexpr int kShortSteps = 4;
template <typename T, int kSeeding, int kW, bool kSample, int kRowWaves>
__global__ void __launch_bounds__(kThreads)
decode_short_kernel(const T* __restrict__ logits, int64_t row_stride, uint32_t V, int64_t B,
                    const int32_t* __restrict__ context, int width, uint64_t key, uint32_t tm1,
                    int none_green, float delta, const uint64_t* __restrict__ seeds, float inv_t,
                    int32_t* __restrict__ tokens, float* __restrict__ values, uint32_t vbase) {
  constexpr int kWaves = kThreads / 64, kRows = kWaves / kRowWaves;
  __shared__ uint64_t lds_key[kWaves], lds_part[kWaves];
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / 64u));
  const uint32_t t = threadIdx.x % (64u * kRowWaves);
  for (int64_t row = static_cast<int64_t>(blockIdx.x) * kRows + wave / kRowWaves; row < B;
       row += static_cast<int64_t>(gridDim.x) * kRows) {
    const T* row_ptr = logits + row * row_stride;
    T raw[kShortSteps];
#pragma unroll
    for (uint32_t n = 0; n < kShortSteps; ++n) {
      const uint32_t c = t + n * 64u * kRowWaves;
      if (c < V) raw[n] = row_ptr[c];
    }
    const RowSeed<kW> rs = row_seed<kSeeding, kW>(key, context + row * width, width);
    const Score<kSample> sc{kSample ? seeds[row] : 0u, inv_t};
    LaneBest best = lane_best_init();
#pragma unroll
    for (uint32_t n = 0; n < kShortSteps; ++n) {
      const uint32_t c = t + n * 64u * kRowWaves;
      if (c < V)
        score_entry<T, kSeeding, kW, kSample>(best, vbase + c, raw_bits(raw[n]), rs, tm1, none_green, delta, sc);
    }
    uint64_t k = best.any ? arg_key(best.v, best.i) : 0u;
    uint64_t p = pack_partial(best.v, best.i);
    wave_argmax(k, p);
    if constexpr (kRowWaves > 1) {
      if (threadIdx.x % 64u == 0u) {
        lds_key[wave] = k;
        lds_part[wave] = p;
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kWaves; ++w)
        if (lds_key[w] > k) { k = lds_key[w]; p = lds_part[w]; }
      __syncthreads();   // the slots are written again for the next row
    }
    if (t == 0u) {
      tokens[row] = static_cast<int32_t>(static_cast<uint32_t>(p));
      if (values != nullptr) values[row] = __uint_as_float(static_cast<uint32_t>(p >> 32));
    }
  }
}

// Read-out: one wavefront per row loads the row's partials at once, reduces their
// keys with shuffles, and lane 0 unpacks the winner.
__global__ void __launch_bounds__(kThreads)
argmax_finish_kernel(const uint64_t* __restrict__ partials, uint32_t segments, int64_t B,
                     int32_t* __restrict__ tokens, float* __restrict__ values) {
  const int lane = threadIdx.x % 64;
  for (int64_t b = static_cast<int64_t>(blockIdx.x) * (kThreads / 64) + threadIdx.x / 64; b < B;
       b += static_cast<int64_t>(gridDim.x) * (kThreads / 64)) {
    const uint64_t* p = partials + b * segments;
    uint64_t bk = 0u, bp = 0u;
    for (uint32_t s = lane; s < segments; s += 64) {
      const uint64_t k = partial_key(p[s]);
      if (k > bk) { bk = k; bp = p[s]; }
    }
    wave_argmax(bk, bp);
    if (lane == 0) {
      tokens[b] = static_cast<int32_t>(static_cast<uint32_t>(bp));
      if (values != nullptr) values[b] = __uint_as_float(static_cast<uint32_t>(bp >> 32));
    }
  }
}

// ---------------------------------------------------------------------------
// Candidate-restricted watermark (top-k self-salt).  One workgroup per row; lane t
// takes candidates t, t + kThreads, ...  A candidate's logit load is issued as soon
// as its id arrives, and the row's window loads, the repeat test and the colour
// draw overlap it.  An id outside [0, V), or equal to an earlier id of the row, is
// skipped, so every logit is written by at most one lane.
// ---------------------------------------------------------------------------
constexpr int kMaxCandidates = 1024;

template <typename T, int kSeeding, int kW>
__global__ void __launch_bounds__(kThreads)
candidates_kernel(T* __restrict__ logits, int64_t row_stride, uint32_t V, int64_t B,
                  const int32_t* __restrict__ cand, int k, const int32_t* __restrict__ context,
                  int width, uint64_t key, uint32_t tm1, float delta) {
  __shared__ int32_t ids[kMaxCandidates];
  for (int64_t row = blockIdx.x; row < B; row += gridDim.x) {
    const int32_t* row_cand = cand + row * k;
    T* row_ptr = logits + row * row_stride;
    for (int j = threadIdx.x; j < k; j += kThreads) ids[j] = row_cand[j];
    const RowSeed<kW> rs = row_seed<kSeeding, kW>(key, context + row * width, width);
    __syncthreads();
    for (int base = 0; base < k; base += kThreads) {
      const int j = base + static_cast<int>(threadIdx.x);
      const int32_t id = j < k ? ids[j] : -1;
      const bool in_range = id >= 0 && static_cast<uint32_t>(id) < V;
      T l{};
      if (in_range) l = row_ptr[id];
      // repeat test: a loop of uniform length over broadcast LDS reads
      const int upto = min(k, base + kThreads) - 1;
      int repeat = 0;
#pragma unroll 8
      for (int i = 0; i < upto; ++i) repeat |= static_cast<int>(ids[i] == id) & static_cast<int>(i < j);
      if (in_range && !repeat && is_green(draw<kSeeding>(rs, static_cast<uint32_t>(id)), tm1))
        row_ptr[id] = bias_elem(l, delta, true);
    }
    __syncthreads();  // ids is refilled for the next row of this workgroup
  }
}

// ---------------------------------------------------------------------------
// Green mask: one lane per 32-bit word (tokens 32w .. 32w+31).
// ---------------------------------------------------------------------------
template <int kSeeding, int kW>
__global__ void __launch_bounds__(kThreads)
green_mask_kernel(uint32_t* __restrict__ bits, uint32_t V, uint32_t words_per_row,
                  const int32_t* __restrict__ context, int width, uint64_t key, uint32_t tm1,
                  int none_green, int64_t num_words) {
  for (int64_t w = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; w < num_words;
       w += static_cast<int64_t>(gridDim.x) * kThreads) {
    const int64_t row = w / words_per_row;
    const uint32_t word = static_cast<uint32_t>(w - row * words_per_row);
    uint32_t out = 0u;
    if (!none_green) {
      const RowSeed<kW> rs = row_seed<kSeeding, kW>(key, context + row * width, width);
      const uint32_t v0 = word * 32u;
      if (kSeeding == kContext) {
        const Key k = key_of(rs.seed);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const Block blk = philox_block(v0 / 4u + q, k);
          const uint32_t xs[4] = {blk.w0, blk.w1, blk.w2, blk.w3};
#pragma unroll
          for (int e = 0; e < 4; ++e)
            out |= static_cast<uint32_t>(is_green(xs[e], tm1)) << (4 * q + e);
        }
      } else {
#pragma unroll 4
        for (int e = 0; e < 32; ++e)
          out |= static_cast<uint32_t>(is_green(draw<kSeeding>(rs, v0 + e), tm1)) << e;
      }
      const uint32_t valid = V - v0;  // >= 1 for every word of the row
      if (valid < 32u) out &= (1u << valid) - 1u;
    }
    bits[w] = out;
  }
}

// ---------------------------------------------------------------------------
// Detect: one wavefront per sequence, ballot + popcount.
// ---------------------------------------------------------------------------
constexpr int kWave = 64;
constexpr int kWavesPerBlock = kThreads / kWave;
constexpr int kMaxSplitWaves = 16;   // most waves of a workgroup that share a sequence

// Lane `l`'s 64-bit value, in every lane.
__device__ __forceinline__ uint64_t readlane64(uint64_t x, int l) {
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(x), l);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(x >> 32), l);
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Lane t gets lane t - 1's x (wave_shr:1); lane 0 gets `first`.
__device__ __forceinline__ uint64_t wave_shift_right(uint64_t x, uint64_t first) {
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
      static_cast<int>(static_cast<uint32_t>(first)), static_cast<int>(static_cast<uint32_t>(x)),
      0x138, 0xF, 0xF, false));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
      static_cast<int>(static_cast<uint32_t>(first >> 32)),
      static_cast<int>(static_cast<uint32_t>(x >> 32)), 0x138, 0xF, 0xF, false));
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Context seeding: membership of token v at a position whose window is w[0..width-1].
template <int kW>
__device__ __forceinline__ bool context_green(uint64_t key, const uint32_t (&w)[kW], int width,
                                              uint32_t v, uint32_t tm1) {
  uint64_t r;
  if constexpr (kW == 1) {
    r = lane_mul_64x32(key, w[0]);
  } else {
    uint64_t sum = 0u;
#pragma unroll
    for (int i = 0; i < kW; ++i)
      if (i < width) sum += w[i];
    r = key * sum;
  }
  return is_green(cbrng_lane(v, r), tm1);
}

// Positions handled per lane per pass: a pass covers 64 * kChunk positions and
// issues all of its token loads before any arithmetic.  The host picks kChunk (see
// detect_plan).
// Outputs of a detect launch; `lengths` (per-sequence token counts, clamped to
// [0, L]) and `scored` (T per sequence) may be null.
struct DetectIO {
  const int32_t* lengths;
  int32_t* counts;
  int32_t* scored;
  double* z;
};

__device__ __forceinline__ int64_t sequence_length(const int32_t* lengths, int64_t n, int64_t L) {
  if (lengths == nullptr) return L;
  const int64_t len = lengths[n];
  return len < 0 ? 0 : (len > L ? L : len);
}

// `shared`: other workgroups have added into the z slot, so the store is atomic as their adds
// are.  The others' is a plain one: written through at device scope it delayed the launch's end
// (4 texts of 20 tokens, context: 2.51 us with it, 2.36 without).
__device__ __forceinline__ void detect_store(const DetectIO& io, int64_t n, uint32_t green,
                                             int64_t T, double gamma, bool shared = false) {
  const double t = static_cast<double>(T);
  const double numerator = static_cast<double>(green) - t * gamma;
  const double denominator = sqrt(t * gamma * (1.0 - gamma));
  io.counts[n] = static_cast<int32_t>(green);
  if (io.scored != nullptr) io.scored[n] = static_cast<int32_t>(T);
  const double z = numerator / denominator;
  if (shared) __hip_atomic_store(&io.z[n], z, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else io.z[n] = z;
}

// One wave's pass: the green positions among base .. base + 64 * kChunk - 1 of a sequence
// of `len` tokens (wave-uniform result; base < len).  Positions are 32-bit (L < 2^31).
// Lanes past the end of the sequence load the last token instead (a valid address), so
// the loads need no branch; their positions are masked out of the count with a lane mask
// built in scalar registers.
//
// Self-salt with a window of several tokens needs K J(w) of every window token: each lane
// computes it once for its own token and the wave shares the products through `kj_lds`
// (kPassTerms entries of its own): position i reads the entries of i - width .. i - 1.
template <int kSeeding, int kW>
constexpr bool kWindowTerms = kSeeding == kSelfSalt && kW > 1;
template <int kChunk>
constexpr int kPassTerms = kMaxWidth + kWave * kChunk;   // the window before the pass, then its tokens

template <int kSeeding, int kChunk, int kW>
__device__ __forceinline__ uint32_t detect_pass(const int32_t* seq, uint32_t base, uint32_t len, int width,
                                                uint64_t key, uint32_t tm1, uint32_t lane,
                                                uint64_t* kj_lds) {
  // The pass's tokens and their windows from two wave-uniform bases; each load adds the
  // lane's byte offset, clamped to the pass's last position.
  const char* pass = reinterpret_cast<const char*>(seq + base);
  const char* pass_w = pass - 4 * width;
  const uint32_t rem = len - base;              // positions left, > 0
  const uint32_t last_byte = 4u * (min(rem, static_cast<uint32_t>(kWave * kChunk)) - 1u);
  uint32_t w[kChunk][kW], v[kChunk];
#pragma unroll
  for (int c = 0; c < kChunk; ++c) {
    const uint32_t ob = min(4u * (static_cast<uint32_t>(c * kWave) + lane), last_byte);
    v[c] = *reinterpret_cast<const uint32_t*>(pass + ob);
#pragma unroll
    for (int k = 0; k < kW; ++k)
      w[c][k] = ((kW == 1 || k < width) && kSeeding == kContext)
                    ? *reinterpret_cast<const uint32_t*>(pass_w + ob + 4u * static_cast<uint32_t>(k))
                    : 0u;
  }
  // Independent membership chains first (instruction-level parallelism), then one ballot
  // per chunk.
  bool g[kChunk];
  if constexpr (kWindowTerms<kSeeding, kW>) {
    uint32_t before = 0u;   // lanes 0 .. width - 1: the window of the pass's first position
    if (lane < static_cast<uint32_t>(width)) before = *reinterpret_cast<const uint32_t*>(pass_w + 4u * lane);
    uint32_t jv[kChunk];
    uint64_t kj[kChunk];
    uint64_t* mine = kj_lds + kMaxWidth + lane;
#pragma unroll
    for (int c = 0; c < kChunk; ++c) {
      jv[c] = jenkins32_lane(v[c]);
      kj[c] = lane_mul_64x32(key, jv[c]);
      mine[c * kWave] = kj[c];
    }
    if (lane < static_cast<uint32_t>(width))
      mine[-width] = lane_mul_64x32(key, jenkins32_lane(before));
    // LDS operations of one wave complete in order; the fences keep the compiler from
    // moving the reads above the writes, or the next pass's writes above these reads.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint64_t* win = mine - width;
#pragma unroll
    for (int c = 0; c < kChunk; ++c) {
      uint64_t r = lane_mul_64x32(kj[c], jv[c]);
#pragma unroll
      for (int k = 0; k < kW; ++k) {
        if (k < width) {
          const uint64_t t = lane_mul_64x32(win[c * kWave + k], jv[c]);
          r = t < r ? t : r;
        }
      }
      g[c] = is_green(cbrng_lane(v[c], r), tm1);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else if constexpr (kSeeding == kSelfSalt) {
    // Self-salt, width 1: the seed of position i is min(K J(p) J(v), K J(v) J(v)) with p
    // the token at i - 1.  Each lane computes K J(v) of its own token once; position i's
    // K J(p) is position i - 1's K J(v), held by the lane before (lane 63 of the chunk
    // before, for lane 0), and a wave shift hands it over.  The pass's first window token
    // is the same for the whole wave: one scalar load, hashed in scalar registers.
    uint32_t jv[kChunk];
    uint64_t kj[kChunk];
#pragma unroll
    for (int c = 0; c < kChunk; ++c) {
      jv[c] = jenkins32_lane(v[c]);
      kj[c] = lane_mul_64x32(key, jv[c]);
    }
    const uint32_t p0 = *reinterpret_cast<const uint32_t*>(pass_w);
    uint64_t carry = key * static_cast<uint64_t>(jenkins32(p0));
#pragma unroll
    for (int c = 0; c < kChunk; ++c) {
      if (c > 0) carry = readlane64(kj[c - 1], kWave - 1);
      const uint64_t kjp = wave_shift_right(kj[c], carry);
      const uint64_t self = lane_mul_64x32(kj[c], jv[c]);
      const uint64_t t = lane_mul_64x32(kjp, jv[c]);
      g[c] = is_green(cbrng_lane(v[c], t < self ? t : self), tm1);
    }
  } else {
#pragma unroll
    for (int c = 0; c < kChunk; ++c) g[c] = context_green<kW>(key, w[c], width, v[c], tm1);
  }
  // Chunks before rem / 64 lie inside the sequence, the next one holds its last rem % 64
  // positions, the others none (masks in scalar registers).
  const uint32_t full_chunks = rem / static_cast<uint32_t>(kWave);
  const uint64_t part_mask = (uint64_t{1} << (rem % static_cast<uint32_t>(kWave))) - 1u;
  uint32_t green = 0u;
#pragma unroll
  for (int c = 0; c < kChunk; ++c) {
    const uint32_t cu = static_cast<uint32_t>(c);
    const uint64_t valid = cu < full_chunks ? ~uint64_t{0} : (cu == full_chunks ? part_mask : 0u);
    green += static_cast<uint32_t>(__popcll(__ballot(g[c]) & valid));
  }
  return green;
}

// Many sequences: one wave each.  The four waves of a workgroup take four sequences;
// their counts meet in LDS and one wave computes the four z-scores side by side (lanes
// 0-3), so the fp64 epilogue issues once per workgroup instead of once per wave.  Every
// wave of the workgroup runs the same number of outer iterations, so the barriers are
// reached by all of them.
template <int kSeeding, int kChunk, int kW>
__global__ void __launch_bounds__(kThreads)
detect_kernel(const int32_t* __restrict__ tokens, int64_t N, int64_t L, int64_t row_stride,
              int width, uint64_t key, uint32_t tm1, double gamma, DetectIO io) {
  __shared__ uint32_t lds_green[kWavesPerBlock], lds_len[kWavesPerBlock];
  __shared__ uint64_t lds_terms[kWindowTerms<kSeeding, kW> ? kWavesPerBlock * kPassTerms<kChunk> : 1];
  const uint32_t lane = threadIdx.x % kWave;
  // the wave's index in the workgroup, in a scalar register
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWave));
  for (int64_t n0 = static_cast<int64_t>(blockIdx.x) * kWavesPerBlock; n0 < N;
       n0 += static_cast<int64_t>(gridDim.x) * kWavesPerBlock) {
    const int64_t n = n0 + wave;
    uint32_t green = 0u;  // wave-uniform count
    uint32_t len = 0u;
    if (n < N) {
      const int32_t* seq = tokens + n * row_stride;
      len = static_cast<uint32_t>(sequence_length(io.lengths, n, L));
      for (uint32_t base = static_cast<uint32_t>(width); base < len; base += kWave * kChunk)
        green += detect_pass<kSeeding, kChunk, kW>(seq, base, len, width, key, tm1, lane,
                                                   lds_terms + wave * kPassTerms<kChunk>);
    }
    if (lane == 0u) {
      lds_green[wave] = green;
      lds_len[wave] = len;
    }
    __syncthreads();
    if (wave == 0 && lane < static_cast<uint32_t>(kWavesPerBlock) && n0 + lane < N) {
      const uint32_t ln = lds_len[lane];
      detect_store(io, n0 + lane, lds_green[lane], ln > static_cast<uint32_t>(width) ? ln - width : 0, gamma);
    }
    __syncthreads();  // the LDS slots are rewritten by the next iteration
  }
}

// Few sequences: the waves of a workgroup (2-16) share one sequence, and `splits`
// workgroups share it too where a sequence is long.  Unit u of the sequence's
// units = splits * waves takes the passes u, u + units, ... of 64 * kChunk positions, so
// texts of any length spread evenly.  With one split the workgroup stores the result.
// With more, the partial counts meet in the sequence's z slot, zeroed by
// detect_zero_kernel before: one 64-bit add carries an arrival (high word) and the green
// count (low word), so the add that brings the last arrival returns all the others'
// counts with it and no fence is needed; that workgroup stores the result over the slot.
template <int kSeeding, int kChunk, int kW>
__global__ void __launch_bounds__(kWave * kMaxSplitWaves)
detect_split_kernel(const int32_t* __restrict__ tokens, int64_t L, int64_t row_stride, int width,
                    uint64_t key, uint32_t tm1, double gamma, uint32_t splits, DetectIO io) {
  __shared__ uint32_t lds_green[kMaxSplitWaves];
  __shared__ uint64_t lds_terms[kWindowTerms<kSeeding, kW> ? kMaxSplitWaves * kPassTerms<kChunk> : 1];
  const uint32_t lane = threadIdx.x % kWave;
  const uint32_t wave =
      static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWave)));
  const uint32_t waves = blockDim.x / kWave;
  const uint32_t n = blockIdx.x / splits;
  const uint32_t split = blockIdx.x % splits;
  const int32_t* seq = tokens + static_cast<int64_t>(n) * row_stride;
  const uint32_t len = static_cast<uint32_t>(sequence_length(io.lengths, n, L));
  constexpr uint32_t kPass = kWave * kChunk;
  const uint32_t step = splits * waves * kPass;
  uint32_t green = 0u;  // wave-uniform count
  for (uint32_t base = static_cast<uint32_t>(width) + (split * waves + wave) * kPass; base < len; base += step)
    green += detect_pass<kSeeding, kChunk, kW>(seq, base, len, width, key, tm1, lane,
                                               lds_terms + wave * kPassTerms<kChunk>);
  if (lane == 0u) lds_green[wave] = green;
  __syncthreads();
  if (threadIdx.x != 0u) return;
  uint32_t sum = 0u;
  for (uint32_t w = 0; w < waves; ++w) sum += lds_green[w];
  if (splits > 1u) {
    uint64_t* slot = reinterpret_cast<uint64_t*>(io.z) + n;
    const uint64_t before = __hip_atomic_fetch_add(slot, (uint64_t{1} << 32) | sum, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
    if (static_cast<uint32_t>(before >> 32) != splits - 1u) return;
    sum += static_cast<uint32_t>(before);
  }
  detect_store(io, n, sum, len > static_cast<uint32_t>(width) ? len - width : 0, gamma, splits > 1u);
}

// Zeroes the z slots that detect_split_kernel adds into.
__global__ void __launch_bounds__(kThreads) detect_zero_kernel(uint64_t* __restrict__ slots, int64_t N) {
  const int64_t n = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
  if (n < N) slots[n] = 0u;
}

// Detection with each distinct (width+1)-gram scored once.  One workgroup per
// sequence: the sequence is staged in LDS, next to an insert-only hash set of
// positions (linear probing; a quarter full, half for the longest texts).  A slot
// holds the position in its low 13 bits and 19 bits of the n-gram's hash above them.
// A lane claims an empty slot with a compare-and-swap, or meets a slot holding an
// equal n-gram and stops there, so exactly one position of every distinct n-gram is
// claimed and scored, whatever the interleaving; the tokens are compared only when
// the hash bits agree.  A position's latency, the chain from hash over probes to draw, bounds
// it, so few texts take many threads (unique_block) and a lane's token is loaded again while
// it probes; two or four positions probed at once per lane measured slower (1024 x 1024:
// 10.4 us with one, 11.1, 12.5).
constexpr uint32_t kMaxUniqueSlots = 8192;   // 32 KB of LDS (+ up to 16 KB of tokens): 4096 positions
constexpr uint32_t kSlotPosBits = 13;        // positions < 8192 (L <= 4096 + kMaxWidth)
constexpr int32_t kEmptySlot = -1;           // never a slot value: no position is 8191
static_assert(kMaxUniqueSlots / 2 + kMaxWidth < (1u << kSlotPosBits) - 1u,
              "every position fits the slot's position bits and differs from 8191");

// Self-salt stages J(token) instead of the token: J is a bijection of 32-bit words (each of
// its steps is), so equal n-grams are those of equal J, and no position hashes its window
// again.  `seq` below holds J(token) (self-salt) or the token (context).
__device__ __forceinline__ uint32_t ngram_hash(const uint32_t* last, int width) {
  // A sum of products with odd constants, then mixed downwards for the slot's low bits.  The
  // multipliers are published ones: 2^32 over the golden ratio (Knuth), MurmurHash3's
  // finaliser (A. Appleby), and a two-round xorshift-multiply hash of C. Wellons' search for
  // integer hashes; any odd ones give the same results.
  uint32_t h = 0u, m = 0x9E3779B1u;
  for (int k = 0; k <= width; ++k) {
    h += last[-k] * m;
    m *= 0x85EBCA6Bu;
  }
  h ^= h >> 15;
  h *= 0x2C1B3C6Du;
  return h ^ (h >> 16);
}

__device__ __forceinline__ bool same_ngram(const uint32_t* a, const uint32_t* b, int width) {
  bool same = true;
  for (int k = 0; k <= width; ++k) same = same && a[-k] == b[-k];
  return same;
}

// Membership of token v, whose staged value is *last, under the window before it.
template <int kSeeding, int kW>
__device__ __forceinline__ bool staged_green(uint64_t key, const uint32_t* last, int width, uint32_t v,
                                             uint32_t tm1) {
  uint64_t r;
  if (kSeeding == kContext) {
    uint64_t sum = 0u;
#pragma unroll
    for (int k = 1; k <= kW; ++k)
      if (kW == 1 || k <= width) sum += last[-k];
    r = kW == 1 ? lane_mul_64x32(key, static_cast<uint32_t>(sum)) : key * sum;
  } else {
    const uint64_t kj = lane_mul_64x32(key, *last);
    r = lane_mul_64x32(kj, *last);
#pragma unroll
    for (int k = 1; k <= kW; ++k) {
      if (kW == 1 || k <= width) {
        const uint64_t t = lane_mul_64x32(kj, last[-k]);
        r = t < r ? t : r;
      }
    }
  }
  return is_green(cbrng_lane(v, r), tm1);
}

constexpr int kStage = 4;   // tokens a lane loads at once when it stages a text
template <int kSeeding, int kW, int kBlock>
__global__ void __launch_bounds__(kBlock)
detect_unique_kernel(const int32_t* __restrict__ tokens, int64_t N, int64_t L, int64_t row_stride,
                     int width, uint64_t key, uint32_t tm1, double gamma, uint32_t slots,
                     DetectIO io) {
  extern __shared__ __attribute__((aligned(16))) int32_t smem[];
  int32_t* table = smem;                                      // `slots` entries, a power of two >= 64
  uint32_t* seq = reinterpret_cast<uint32_t*>(smem + slots);  // the staged sequence (up to L)
  __shared__ uint32_t sums[2];
  for (int64_t n = blockIdx.x; n < N; n += gridDim.x) {
    const int32_t* src = tokens + n * row_stride;
    const int len = static_cast<int>(sequence_length(io.lengths, n, L));   // at most 4096 + kMaxWidth
    for (int t0 = threadIdx.x; t0 < len; t0 += kStage * kBlock) {
      uint32_t v[kStage];
#pragma unroll
      for (int u = 0; u < kStage; ++u) v[u] = static_cast<uint32_t>(src[min(t0 + u * kBlock, len - 1)]);
#pragma unroll
      for (int u = 0; u < kStage; ++u)
        if (t0 + u * kBlock < len) seq[t0 + u * kBlock] = kSeeding == kSelfSalt ? jenkins32_lane(v[u]) : v[u];
    }
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    for (uint32_t sl = 4u * threadIdx.x; sl < slots; sl += 4u * kBlock)
      *reinterpret_cast<i32x4*>(table + sl) = i32x4{kEmptySlot, kEmptySlot, kEmptySlot, kEmptySlot};
    if (threadIdx.x < 2) sums[threadIdx.x] = 0u;
    __syncthreads();
    uint32_t trials = 0u, green = 0u;   // of the wave (the same in every lane)
    // a wave's first position decides whether it takes the pass: all its lanes go along
    for (int base = width + static_cast<int>(threadIdx.x & ~63u); base < len; base += kBlock) {
      const int i = min(base + static_cast<int>(threadIdx.x % 64u), len - 1);
      const uint32_t* last = seq + i;
      const uint32_t v = kSeeding == kSelfSalt ? static_cast<uint32_t>(src[i]) : *last;   // arrives while the lane probes
      const uint32_t h = ngram_hash(last, width);
      constexpr uint32_t kPos = (1u << kSlotPosBits) - 1u;
      const uint32_t mine = (h & ~kPos) | static_cast<uint32_t>(i);
      uint32_t slot = h & (slots - 1u);
      bool looking = base + static_cast<int>(threadIdx.x % 64u) < len, claimed = false;
      // at most `slots` probes; the set never fills, so a lane stops long before
      for (uint32_t probe = 0; probe < slots; ++probe) {
        if (looking) {
          const uint32_t held = static_cast<uint32_t>(atomicCAS(&table[slot], kEmptySlot, static_cast<int32_t>(mine)));
          claimed = held == static_cast<uint32_t>(kEmptySlot);
          looking = !claimed && !((held & ~kPos) == (mine & ~kPos) && same_ngram(seq + (held & kPos), last, width));
          slot = (slot + 1u) & (slots - 1u);
        }
        if (!__any(looking)) break;
      }
      trials += static_cast<uint32_t>(__popcll(__ballot(claimed)));
      bool g = false;
      if (claimed) g = staged_green<kSeeding, kW>(key, last, width, v, tm1);
      green += static_cast<uint32_t>(__popcll(__ballot(g)));
    }
    if (threadIdx.x % 64 == 0) {
      atomicAdd(&sums[0], trials);
      atomicAdd(&sums[1], green);
    }
    __syncthreads();
    if (threadIdx.x == 0) detect_store(io, n, sums[1], sums[0], gamma);
    __syncthreads();  // the table and sums are reset for the next sequence
  }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
thread_local hipError_t g_last_hip_error = hipSuccess;

// ceil(gamma * 2^32) clamped to [0, 2^32] (the scaling by 2^32 is exact).
uint64_t threshold_of(double gamma) {
  const double scaled = ceil(gamma * 4294967296.0);
  if (!(scaled > 0.0)) return 0u;
  if (scaled >= 4294967296.0) return 4294967296ull;
  return static_cast<uint64_t>(scaled);
}

sbw_status_t check_device() {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) {
    g_last_hip_error = e;
    (void)hipGetLastError();
    return SBW_ERR_NO_DEVICE;
  }
  return SBW_OK;
}

sbw_status_t after_launch() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    g_last_hip_error = e;
    return SBW_ERR_HIP;
  }
  return SBW_OK;
}

int64_t grid_for(int64_t work_groups) { return work_groups < kMaxGrid ? work_groups : kMaxGrid; }

bool valid_seeding(int s) { return s == SBW_SEED_CONTEXT || s == SBW_SEED_SELF_SALT; }

sbw_status_t check_width(int64_t width) {
  if (width < 1) return SBW_ERR_INVALID_ARG;
  if (width > kMaxWidth) return SBW_ERR_UNSUPPORTED;
  return SBW_OK;
}

// Self-salt row kernel: one quad per lane below this many workgroups of two (B = 64 rows
// of 19008, 640 workgroups: 5.6 us either way at width 4, 4.6 / 5.0 with one / two at width
// 1; 16 rows of 128256, 1008: 7.5 / 6.9 us at width 4).
constexpr int64_t kTwoQuadMinGroups = 960;

// Rows that a workgroup of the self-salt row kernel takes in turn with the candidate terms
// of its columns computed once.  A row costs 1, the terms a third of one; a CU runs its
// share of the workgroups side by side at a fixed rate, so a launch takes as long as the
// CU with the most: ceil(workgroups / 256) * (rows + 1/3).  The least of it over 1-8 rows
// with at least 4 workgroups for most CUs (fewer leave latency bare).  Width 4 fp32, rows
// 1 / 2 / 3 / 4: 64 x 151936 26.9 / 25.0 / 24.1 / 23.4 us, 128 x 50000 18.7 / 17.8 / 18.5 /
// 19.6 us, 256 x 152064 (1 / 4 / 6 / 8) 99.0 / 85.8 / 83.9 / 87.0 us.
int64_t rows_per_slot(int64_t tiles, int64_t B) {
  int64_t best = 1, best_cost = INT64_MAX;
  for (int64_t rows = 1; rows <= 8; ++rows) {
    const int64_t groups = tiles * ((B + rows - 1) / rows);
    if (rows > 1 && groups < kTwoQuadMinGroups) break;
    const int64_t cost = (groups + 255) / 256 * (3 * rows + 1);
    if (cost < best_cost) {
      best = rows;
      best_cost = cost;
    }
  }
  return best;
}

// Whether a launch takes one token per lane: rows of at most a workgroup's lanes, where vectors
// would leave most of it idle (5000 x 100 fp32, context: 4.7 us, 6.7 with vectors), and small
// launches.  The lines for these, where the two cross: rows of whole vectors 256K logits, fewer
// with the wider windows of self-salt, whose shared terms are worth more (context fp32 256K
// logits 2.25-2.34 us, vectors 2.32, 384K 2.5 / 2.4; self-salt width 2 192K 2.5 / 2.55, 256K
// 2.7 / 2.6; width 4 128K 2.55 / 2.72, 192K 2.83 / 2.78; width 8 128K 3.1 / 3.1).  Rows with edge
// columns, whose workgroups cost vectors about 0.5 us: context 300K 2.9-3.0 / 2.93-3.07, 400K
// 3.1-3.3 / 3.0-3.1; width 1 400K 3.3 / 3.5, 500K 3.8 / 3.6; width 2 400K 3.6 / 3.6; width 4 300K
// 3.7 / 3.7; width 8 150K 3.86 / 3.90, 200K 4.2 / 3.9; twice as many where such a row is shorter
// than a tile (1300 x 301, width 1: 4.0 / 5.2; 1000 x 401, width 4: 4.6 / 5.1).
template <int kSeeding, int kW>
bool one_token_a_lane(int64_t B, uint32_t V, bool edges) {
  constexpr int64_t kWhole = kSeeding == kContext || kW == 1 ? 8 : kW == 2 ? 6 : kW <= kMidWidth ? 5 : 4;
  constexpr int64_t kEdges = kSeeding == kContext ? 10 : kW == 1 ? 13 : kW == 2 ? 12 : kW <= kMidWidth ? 9 : 5;
  const int64_t most = edges ? kEdges << (V <= 2 * kThreads ? 16 : 15) : kWhole << 15;
  return V <= kThreads || B <= most / V;
}

template <typename T, int kSeeding, int kW>
void launch_watermark(void* logits, int64_t B, uint32_t V, int64_t row_stride,
                      const int32_t* context, int width, uint64_t key, uint32_t tm1, float delta,
                      uint32_t vbase, hipStream_t stream) {
  T* p = static_cast<T*>(logits);
  const uint32_t rows = static_cast<uint32_t>(B < kMaxGridY ? B : kMaxGridY);
  const RowSplit split = row_split<kSeeding == kSelfSalt ? 4u : 16u / sizeof(T)>(V, vbase);
  if (one_token_a_lane<kSeeding, kW>(B, V, split.head + split.tail != 0u)) {
    const uint32_t threads = V < kThreads ? (V + 63u) / 64u * 64u : kThreads;
    hipLaunchKernelGGL((watermark_token_kernel<T, kSeeding, kW>), dim3((V + threads - 1) / threads, rows),
                       dim3(threads), 0, stream, p, row_stride, V, B, context, width, key, tm1, delta, vbase);
    return;
  }
  constexpr uint32_t kPer = 16u / sizeof(T);
  const RowSplit sp = row_split<kPer>(V, vbase);
  const uint64_t vectors = sp.full;
  // grid rows for the edge columns, and those that `most` rows of tiles take beside them
  auto edge_rows = [&](const RowSplit& r, uint32_t tiles) -> uint32_t {
    if (r.head + r.tail == 0u) return 0u;
    const int64_t groups = (B + kEdgeRows - 1) / kEdgeRows;
    const int64_t y = (groups + tiles - 1) / tiles;
    return static_cast<uint32_t>(y < kMaxEdgeY ? y : kMaxEdgeY);
  };
  auto slots_of = [&](int64_t most, uint32_t edge_y) {
    return static_cast<uint32_t>(most < kMaxGridY - edge_y ? most : kMaxGridY - edge_y);
  };
  if constexpr (kSeeding == kSelfSalt) {
    if constexpr (kW == 1) {
      const uint32_t tiles1 = static_cast<uint32_t>((vectors + kThreads - 1) / kThreads);
      auto launch_slab = [&](auto height) -> bool {
        constexpr int kRows = decltype(height)::value;
        const int64_t slabs = (B + kRows - 1) / kRows;
        const int64_t least = kRows == 12      ? SBW_SLAB12_MIN_GROUPS
                              : sizeof(T) == 2 ? SBW_SLAB_BF16_MIN_GROUPS : SBW_SLAB_MIN_GROUPS;
        if (static_cast<int64_t>(tiles1) * slabs < least) return false;
        const uint32_t edge_y = edge_rows(sp, tiles1);
        const uint32_t slots = slots_of(slabs, edge_y);
        const dim3 grid(tiles1, slots + edge_y);
        if (edge_y != 0u)
          hipLaunchKernelGGL((watermark_ss_slab_kernel<T, kRows, true>), grid, dim3(kThreads), 0, stream, p,
                             row_stride, V, B, context, key, tm1, delta, vbase, slots);
        else
          hipLaunchKernelGGL((watermark_ss_slab_kernel<T, kRows, false>), grid, dim3(kThreads), 0, stream, p,
                             row_stride, V, B, context, key, tm1, delta, vbase, slots);
        return true;
      };
      if (launch_slab(std::integral_constant<int, 12>{})) return;
      if (launch_slab(std::integral_constant<int, 8>{})) return;
      if constexpr (sizeof(T) == 4) {
        if (launch_slab(std::integral_constant<int, 6>{})) return;
      }
    }
    const RowSplit quads = row_split<4>(V, vbase);
    const uint32_t tiles2 = (quads.full + 2 * kThreads - 1) / (2 * kThreads);
    if (tiles2 * B < kTwoQuadMinGroups) {
      const uint32_t tiles = (quads.full + kThreads - 1) / kThreads;
      const uint32_t edge_y = edge_rows(quads, tiles), slots = slots_of(B, edge_y);
      if (edge_y != 0u)
        hipLaunchKernelGGL((watermark_ss_rows_kernel<T, 1, kW, true>), dim3(tiles, slots + edge_y), dim3(kThreads),
                           0, stream, p, row_stride, V, B, context, key, tm1, delta, vbase, slots);
      else
        hipLaunchKernelGGL((watermark_ss_rows_kernel<T, 1, kW, false>), dim3(tiles, slots + edge_y), dim3(kThreads),
                           0, stream, p, row_stride, V, B, context, key, tm1, delta, vbase, slots);
      return;
    }
    const uint32_t edge_y = edge_rows(quads, tiles2);
    const uint32_t slots = slots_of((B + rows_per_slot(tiles2, B) - 1) / rows_per_slot(tiles2, B), edge_y);
    if (edge_y != 0u)
      hipLaunchKernelGGL((watermark_ss_rows_kernel<T, 2, kW, true>), dim3(tiles2, slots + edge_y), dim3(kThreads),
                         0, stream, p, row_stride, V, B, context, key, tm1, delta, vbase, slots);
    else
      hipLaunchKernelGGL((watermark_ss_rows_kernel<T, 2, kW, false>), dim3(tiles2, slots + edge_y), dim3(kThreads),
                         0, stream, p, row_stride, V, B, context, key, tm1, delta, vbase, slots);
  } else {
    // Two vectors in flight per lane measured best (~80 % of HBM peak; one: ~75 %).
    constexpr int kU = sizeof(T) == 4 ? SBW_CONTEXT_UNROLL : SBW_CONTEXT_UNROLL_BF16;
    const uint32_t tiles = static_cast<uint32_t>((vectors + kThreads * kU - 1) / (kThreads * kU));
    // whole rows per XCD for large launches (one launch row per grid row, workgroup
    // numbers below 2^32)
    const uint32_t edge_y = edge_rows(sp, tiles);
    const bool spread = edge_y != 0u && B >= kSpreadRows;
    // spread: the rarest grid rows that are enough for the edges, rows / (2^shift - 1) of them
    // (every second one at most; each takes more rows in turn where that is too few)
    uint32_t shift = 1u;
    while (spread && rows / ((uint64_t{2} << shift) - 1) >= edge_y) ++shift;
    const uint64_t every = (uint64_t{1} << shift) - 1;
    const uint64_t grid_rows = spread ? rows + (rows + every - 1) / every : uint64_t{rows} + edge_y;
    const uint32_t xcd_rows =
        B >= SBW_XCD_ROWS_MIN && B % 8 == 0 && grid_rows <= kMaxGridY &&
                B * static_cast<int64_t>(V) * static_cast<int64_t>(sizeof(T)) >= SBW_XCD_ROWS_MIN_BYTES &&
                uint64_t{tiles} * grid_rows < (uint64_t{1} << 32)
            ? 1u
            : 0u;
    const uint32_t slots = slots_of(B, edge_y);
    const dim3 grid(tiles, spread ? static_cast<uint32_t>(grid_rows < kMaxGridY ? grid_rows : kMaxGridY)
                                  : slots + edge_y);
    if (spread)
      hipLaunchKernelGGL((watermark_vec_kernel<T, kU, kW, true>), grid, dim3(kThreads), 0, stream, p, row_stride,
                         V, B, context, width, key, tm1, delta, vbase, xcd_rows, shift);
    else
      hipLaunchKernelGGL((watermark_vec_kernel<T, kU, kW, false>), grid, dim3(kThreads), 0, stream, p, row_stride,
                         V, B, context, width, key, tm1, delta, vbase, xcd_rows, slots);
  }
}

template <typename T>
void dispatch_watermark(void* logits, int64_t B, uint32_t V, int64_t row_stride,
                        const int32_t* context, int width, uint64_t key, uint32_t tm1, float delta,
                        sbw_seeding_t seeding, uint32_t vbase, hipStream_t st) {
  // Context seeding folds any window into one row seed; self-salt needs the window per
  // candidate and has an instantiation for each width.
  if (seeding == SBW_SEED_CONTEXT)
    launch_watermark<T, kContext, kMaxWidth>(logits, B, V, row_stride, context, width, key, tm1,
                                             delta, vbase, st);
  else {
    auto launch = [&](auto w) {
      launch_watermark<T, kSelfSalt, decltype(w)::value>(logits, B, V, row_stride, context, width, key,
                                                         tm1, delta, vbase, st);
    };
    switch (width) {
      case 1: launch(std::integral_constant<int, 1>{}); break;
      case 2: launch(std::integral_constant<int, 2>{}); break;
      case 3: launch(std::integral_constant<int, 3>{}); break;
      case 4: launch(std::integral_constant<int, 4>{}); break;
      case 5: launch(std::integral_constant<int, 5>{}); break;
      case 6: launch(std::integral_constant<int, 6>{}); break;
      case 7: launch(std::integral_constant<int, 7>{}); break;
      default: launch(std::integral_constant<int, 8>{}); break;
    }
  }
}

template <typename T>
void dispatch_candidates(void* logits, int64_t B, uint32_t V, int64_t row_stride,
                         const int32_t* cand, int k, const int32_t* context, int width,
                         uint64_t key, uint32_t tm1, float delta, sbw_seeding_t seeding,
                         hipStream_t st) {
  T* p = static_cast<T*>(logits);
  const dim3 grid(static_cast<uint32_t>(grid_for(B)));
  if (seeding == SBW_SEED_CONTEXT)
    hipLaunchKernelGGL((candidates_kernel<T, kContext, kMaxWidth>), grid, dim3(kThreads), 0, st, p,
                       row_stride, V, B, cand, k, context, width, key, tm1, delta);
  else if (width == 1)
    hipLaunchKernelGGL((candidates_kernel<T, kSelfSalt, 1>), grid, dim3(kThreads), 0, st, p,
                       row_stride, V, B, cand, k, context, width, key, tm1, delta);
  else if (width <= kMidWidth)
    hipLaunchKernelGGL((candidates_kernel<T, kSelfSalt, kMidWidth>), grid, dim3(kThreads), 0, st,
                       p, row_stride, V, B, cand, k, context, width, key, tm1, delta);
  else
    hipLaunchKernelGGL((candidates_kernel<T, kSelfSalt, kMaxWidth>), grid, dim3(kThreads), 0, st,
                       p, row_stride, V, B, cand, k, context, width, key, tm1, delta);
}

// Vectors per lane (and so segments per row) of the fused decoding.
template <typename T>
constexpr int decode_vecs_for(bool sample) {
  return sizeof(T) == 4 ? (sample ? SBW_DECODE_VECS_F32 : SBW_DECODE_VECS_F32_GREEDY)
                        : (sample ? SBW_DECODE_VECS_BF16_SAMPLE : SBW_DECODE_VECS_BF16);
}
template <typename T>
constexpr int decode_subs_for(bool sample) { return sizeof(T) == 2 && !sample ? SBW_DECODE_SUBS_BF16 : 1; }
template <typename T>
constexpr uint64_t vec_segment_elems(int kN) { return (16u / sizeof(T)) * kThreads * kN; }
// Small grids: a launch of fewer workgroups than this takes half the vectors per lane
// (twice the segments), which hides more of the load latency when the chip is not
// full: a vocabulary shard of 19008 fp32 or bf16 logits at B = 256 gets 1280
// workgroups instead of 768 (about 8 % faster); B = 64 rows of 152064 (960-1600
// workgroups) stay.  Such a launch takes them in one sub-batch: with few waves in flight a
// second one only adds its bounds and test (greedy bf16, rows of 128256, two / one: B = 1
// 5.37 / 5.26 us, B = 32 6.95 / 6.75, N(0,1) logits 9.27 / 8.80).
constexpr int64_t kSmallDecodeGrid = 900;
// The workspace is sized for segments of kArgmaxSegElems; none may be shorter.
static_assert(vec_segment_elems<float>(SBW_DECODE_VECS_F32 / 2) >= kArgmaxSegElems &&
                  vec_segment_elems<float>(SBW_DECODE_VECS_F32_GREEDY / 2) >= kArgmaxSegElems &&
                  vec_segment_elems<uint16_t>(SBW_DECODE_VECS_BF16 / 2) >= kArgmaxSegElems &&
                  SBW_DECODE_VECS_BF16 % SBW_DECODE_SUBS_BF16 == 0 &&
                  vec_segment_elems<uint16_t>(SBW_DECODE_VECS_BF16_SAMPLE / 2) >= kArgmaxSegElems,
              "the segments of a row must fit its part of the workspace");

// The per-row noise seeds and 1/T of a sampling pass (unused by greedy decoding).
struct SampleArgs {
  const uint64_t* seeds;
  float inv_t;
};

// The longest rows for the short kernel, and of launches of up to kShortCells logits: with
// many longer rows the tokens that the segment pass leaves undrawn are worth more than its
// fixed part (self-salt greedy fp32, 5000 x 513 14.3 us in segments, 13.4 here, x 1001 14.8 /
// 17.5; 1000 x 1001 6.7 / 5.6).
constexpr uint32_t kShortRow = 640, kShortRowFew = 1024;
constexpr int64_t kShortCells = int64_t{1} << 20;
static_assert(kShortRowFew <= kThreads * kShortSteps, "a workgroup holds a short row");

template <typename T, int kSeeding, int kW, bool kSample>
void launch_argmax(const void* logits, int64_t B, uint32_t V, int64_t row_stride,
                   const int32_t* context, int width, uint64_t key, uint32_t tm1, int none,
                   float delta, const SampleArgs& sa, uint32_t vbase, int32_t* tokens, float* values,
                   uint64_t* partials, hipStream_t stream) {
  const T* p = static_cast<const T*>(logits);
  const uint32_t rows = static_cast<uint32_t>(B < kMaxGridY ? B : kMaxGridY);
  if (V <= kShortRow || (V <= kShortRowFew && B <= kShortCells / V)) {
    auto launch_short = [&](auto row_waves) {
      constexpr int kRowWaves = decltype(row_waves)::value;
      constexpr int kRows = kThreads / 64 / kRowWaves;
      hipLaunchKernelGGL((decode_short_kernel<T, kSeeding, kW, kSample, kRowWaves>),
                         dim3(static_cast<uint32_t>(grid_for((B + kRows - 1) / kRows))), dim3(kThreads), 0,
                         stream, p, row_stride, V, B, context, width, key, tm1, none, delta, sa.seeds,
                         sa.inv_t, tokens, values, vbase);
    };
    // one wave a row where the rows fill the chip or one step holds them (1000 x 256 greedy 3.2
    // us, 3.6 with four waves; 64 x 256 sampling 4.1 / 3.2)
    if (V <= 64u || (V <= 64u * kShortSteps && B >= 512)) launch_short(std::integral_constant<int, 1>{});
    else launch_short(std::integral_constant<int, kThreads / 64>{});
    return;
  }
  constexpr int kSub = decode_subs_for<T>(kSample);
  constexpr int kN = decode_vecs_for<T>(kSample) / kSub;
  constexpr int kNs = kN * kSub / 2;
  const bool crowded = sizeof(T) == 4 && !kSample &&
                       B * static_cast<int64_t>(V) * 4 >= SBW_XCD_ROWS_MIN_BYTES;
  const uint32_t spare_lds = crowded ? kCrowdedLds : 0u;
  auto launch = [&](auto vecs, auto subs, uint64_t seg) {
    const uint32_t segments = static_cast<uint32_t>((uint64_t{V} + seg - 1) / seg);
    hipLaunchKernelGGL((decode_vec_kernel<T, kSeeding, decltype(vecs)::value, decltype(subs)::value, kW, kSample>),
                       dim3(segments, rows), dim3(kThreads), spare_lds, stream, p, row_stride, V, B, context,
                       width, key, tm1, none, delta, sa.seeds, sa.inv_t, segments, partials, vbase);
    return segments;
  };
  const uint64_t seg = vec_segment_elems<T>(kN) * kSub;
  uint32_t segments;
  if ((V + static_cast<int64_t>(seg) - 1) / static_cast<int64_t>(seg) * rows >= kSmallDecodeGrid)
    segments = launch(std::integral_constant<int, kN>{}, std::integral_constant<int, kSub>{}, seg);
  else
    segments = launch(std::integral_constant<int, kNs>{}, std::integral_constant<int, 1>{},
                      vec_segment_elems<T>(kNs));
  const int64_t row_blocks = grid_for((B + kThreads / 64 - 1) / (kThreads / 64));
  hipLaunchKernelGGL(argmax_finish_kernel, dim3(row_blocks), dim3(kThreads), 0, stream, partials,
                     segments, B, tokens, values);
}

template <typename T, bool kSample>
void dispatch_argmax(const void* logits, int64_t B, uint32_t V, int64_t row_stride,
                     const int32_t* context, int width, uint64_t key, uint32_t tm1, int none,
                     float delta, const SampleArgs& sa, sbw_seeding_t seeding, uint32_t vbase,
                     int32_t* tokens, float* values, uint64_t* partials,
                     hipStream_t st) {
  if (seeding == SBW_SEED_CONTEXT)
    launch_argmax<T, kContext, kMaxWidth, kSample>(logits, B, V, row_stride, context, width, key,
                                                   tm1, none, delta, sa, vbase, tokens,
                                                   values, partials, st);
  else if (width == 1)
    launch_argmax<T, kSelfSalt, 1, kSample>(logits, B, V, row_stride, context, width, key, tm1,
                                            none, delta, sa, vbase, tokens, values,
                                            partials, st);
  else if (width <= kMidWidth)
    launch_argmax<T, kSelfSalt, kMidWidth, kSample>(logits, B, V, row_stride, context, width, key,
                                                    tm1, none, delta, sa, vbase, tokens,
                                                    values, partials, st);
  else
    launch_argmax<T, kSelfSalt, kMaxWidth, kSample>(logits, B, V, row_stride, context, width, key,
                                                    tm1, none, delta, sa, vbase, tokens,
                                                    values, partials, st);
}

// How a detect launch spreads over the chip: waves and workgroups per sequence, positions
// per lane and pass.  All times per launch, 100-launch graphs, one box (start = one wave
// per sequence, 8 chunks a pass).
//  * A wave per sequence (detect_kernel) where the sequences alone fill the chip: above
//    1024 of them with a window of one token (N = 2048, L = 512, context: 4.3 us against
//    4.8 with 4 waves), above 2048 with wider windows (N = 2048, L = 512 / 1024, width 4:
//    context 5.5 / 7.8 us with 4 waves against 7.0 / 11.2); and where a sequence has too few
//    chunks for the sharing to pay: two from 256 sequences (N = 1000, L = 80, context 2.64 us,
//    2.92 with two waves), width 1 also three (N = 500, L = 180, 2.9 / 3.0) and, from 768, four
//    (N = 1000, L = 250, self-salt 3.28 / 3.43).  Chunks per pass: the most that pad a sequence
//    by at most a sixth (N = 16384, L = 300, self-salt: 15.2 us with one chunk, 20.8 with 8;
//    N = 4096, L = 512: 7.7 against 7.1 the other way), a third up to 2048 sequences, whose
//    waves the chip holds at once (N = 2000, L = 400, self-salt: 5.9 us with one, 4.9 with 8).
//  * Otherwise up to 16 waves share a sequence, as many as keep 8192 waves in all and one
//    chunk each (from 512 sequences as few as leave each at most two: N = 1024, L = 512,
//    self-salt 4.0 us, one each 4.2; L = 300, width 4, two or three each 4.7, at most two 4.3);
//    two chunks a pass where a wave has them.  N = 128, L = 2048, self-salt width 4: 19.6 ->
//    4.5 us.
//  * Longer than 64 chunks, 8-wave workgroups split a sequence, splits^2 * N <= 2048:
//    more splits cost more in adds to one slot than they save, and the zeroing launch
//    costs about 2 us (N = 32, L = 4096: 5.1 us unsplit, 5.4 split; L = 16384: 122 -> 7.0).
//    N = 8, L = 16384, context width 4: 121 us at the start, 6.1 now.
//  * Context seeding with a wide window takes one chunk a pass throughout: the window's
//    loads of several chunks in flight cost more than they hide (N = 4096, L = 512,
//    width 4: 7.8 us, with 8 chunks 9.2).
struct DetectPlan {
  int waves, chunk;
  uint32_t splits;   // 0: detect_kernel, one wave per sequence
};

template <int kSeeding, int kW>
constexpr int kMaxDetectChunk = kSeeding == kContext && kW > 1 ? 1 : (kW > kMidWidth ? 4 : 8);

template <int kSeeding, int kW>
DetectPlan detect_plan(int64_t N, int64_t positions) {
  constexpr int kMaxChunk = kMaxDetectChunk<kSeeding, kW>;
  const int64_t chunks = (positions + kWave - 1) / kWave;
  if (N > (kW == 1 ? 1024 : 2048) || chunks < 2 || (N >= 256 && chunks <= (kW == 1 ? 3 : 2)) ||
      (kW == 1 && N >= 768 && chunks <= 4)) {
    int chunk = kMaxChunk;
    const int64_t slack = N <= 2048 ? 3 : 6;
    while (chunk > 1 && ((chunks + chunk - 1) / chunk * chunk - chunks) * slack > chunks) chunk /= 2;
    return DetectPlan{1, chunk, 0u};
  }
  DetectPlan p{kMaxSplitWaves, 1, 1u};
  if (chunks > 64) {
    while (p.splits * 16 <= chunks && 4 * int64_t{p.splits} * p.splits * N <= 2048) p.splits *= 2;
    if (p.splits > 1u) p.waves = 8;
  }
  const int64_t each = kMaxChunk > 1 && N >= 512 ? 2 : 1;   // chunks that a wave has at most
  while (p.waves > 1 && (p.waves * N > 8192 || p.waves / 2 * each >= chunks)) p.waves /= 2;
  if (kMaxChunk > 1 && 2 * p.waves * int64_t{p.splits} <= chunks) p.chunk = 2;
  return p;
}

template <int kSeeding, int kW>
void launch_detect(int64_t positions, hipStream_t st, const int32_t* tokens, int64_t N, int64_t L,
                   int64_t row_stride, int width, uint64_t key, uint32_t tm1, double gamma,
                   const DetectIO& io) {
  constexpr int kMaxChunk = kMaxDetectChunk<kSeeding, kW>;
  const DetectPlan plan = detect_plan<kSeeding, kW>(N, positions);
  if (plan.splits == 0u) {
    const dim3 grid(static_cast<uint32_t>(grid_for((N + kWavesPerBlock - 1) / kWavesPerBlock)));
    auto launch = [&](auto chunk) {
      constexpr int kChunk = decltype(chunk)::value <= kMaxChunk ? decltype(chunk)::value : kMaxChunk;
      hipLaunchKernelGGL((detect_kernel<kSeeding, kChunk, kW>), grid, dim3(kThreads), 0, st, tokens, N,
                         L, row_stride, width, key, tm1, gamma, io);
    };
    if (plan.chunk == 1) launch(std::integral_constant<int, 1>{});
    else if (plan.chunk == 2) launch(std::integral_constant<int, 2>{});
    else if (plan.chunk == 4) launch(std::integral_constant<int, 4>{});
    else launch(std::integral_constant<int, 8>{});
    return;
  }
  if (plan.splits > 1u)
    hipLaunchKernelGGL(detect_zero_kernel, dim3(static_cast<uint32_t>((N + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, st, reinterpret_cast<uint64_t*>(io.z), N);
  auto launch = [&](auto chunk) {
    constexpr int kChunk = decltype(chunk)::value <= kMaxChunk ? decltype(chunk)::value : kMaxChunk;
    hipLaunchKernelGGL((detect_split_kernel<kSeeding, kChunk, kW>),
                       dim3(static_cast<uint32_t>(N) * plan.splits), dim3(kWave * plan.waves), 0, st,
                       tokens, L, row_stride, width, key, tm1, gamma, plan.splits, io);
  };
  if (plan.chunk == 1) launch(std::integral_constant<int, 1>{});
  else launch(std::integral_constant<int, 2>{});
}

// Threads of the workgroup that takes a text with the repeat rule: the most that its
// positions keep busy while the launch stays within 4096 waves, as every text costs its waves'
// launch, staging and barriers (about 1.6 waves start per ns); but enough for 24 waves a CU
// where the texts' LDS lets only few workgroups share one, 16 up to 1024 texts, which leave a
// CU four at most (1024 x 1040, context: 9.0 us, 9.7 with 512 threads).  us at 64 / 128 / 256 / 512 threads
// (1024 for the last three): 4000 texts of 60 tokens 6.0 / 7.5 / 10.3 / 19.1; 4096 x 512 20.5 /
// 15.2 / 16.1 / 21.3; 8000 x 1000 75 / 49 / 38 / 52; 1024 x 1024 25.1 / 15.3 / 11.0 / 11.7;
// 512 x 512 11.4 / 7.4 / 5.7 / 5.1; 512 x 4096 140 / 81 / 45 / 31.7 (36); 256 x 1024 24.0 / 14.0 /
// 9.0 / 6.9 (6.3); 16 x 4096 96 / 52 / 29.5 / 18.8 (14.0).  Before: 256 for every text, 29.6 us
// for 16 x 4096.
int unique_block(int64_t N, int64_t positions, size_t lds) {
  int block = 64;
  while (block < 1024 && block < positions &&
         (N * 2 * block <= 64 * 4096 ||
          static_cast<size_t>(block) * 160 * 1024 < 64 * (N > 1024 ? 24 : 16) * lds))
    block *= 2;
  return block;
}

template <int kSeeding, int kW>
void launch_detect_unique(int64_t N, hipStream_t st, const int32_t* tokens, int64_t L,
                          int64_t row_stride, int width, uint64_t key, uint32_t tm1, double gamma,
                          uint32_t slots, const DetectIO& io) {
  const size_t lds = (static_cast<size_t>(slots) + static_cast<size_t>(L)) * sizeof(int32_t);
  auto launch = [&](auto block) {
    constexpr int kBlock = decltype(block)::value;
    hipLaunchKernelGGL((detect_unique_kernel<kSeeding, kW, kBlock>), dim3(static_cast<uint32_t>(grid_for(N))),
                       dim3(kBlock), lds, st, tokens, N, L, row_stride, width, key, tm1, gamma, slots, io);
  };
  const int block = unique_block(N, L - width, lds);
  if (block == 64) launch(std::integral_constant<int, 64>{});
  else if (block == 128) launch(std::integral_constant<int, 128>{});
  else if (block == 256) launch(std::integral_constant<int, 256>{});
  else if (block == 512) launch(std::integral_constant<int, 512>{});
  else launch(std::integral_constant<int, 1024>{});
}

// Every detect entry point: validation, then one launch.
sbw_status_t detect_impl(const int32_t* tokens, int64_t N, int64_t L, int64_t row_stride,
                         const int32_t* lengths, int64_t width, uint64_t key, double gamma,
                         sbw_seeding_t seeding, uint32_t flags, int32_t* green_counts,
                         int32_t* scored, double* z, hipStream_t st) {
  if (N < 0 || L < 0 || row_stride < L) return SBW_ERR_INVALID_ARG;
  sbw_status_t s = check_width(width);
  if (s != SBW_OK) return s;
  if (!valid_seeding(seeding)) return SBW_ERR_UNSUPPORTED;
  if ((flags & ~static_cast<uint32_t>(SBW_DETECT_IGNORE_REPEATED)) != 0u) return SBW_ERR_UNSUPPORTED;
  if (!(gamma > 0.0 && gamma < 1.0)) return SBW_ERR_GAMMA;
  if (L > INT32_MAX) return SBW_ERR_UNSUPPORTED;
  const bool unique = (flags & SBW_DETECT_IGNORE_REPEATED) != 0u;
  const int64_t positions = L > width ? L - width : 0;
  if (unique && 2 * positions > static_cast<int64_t>(kMaxUniqueSlots)) return SBW_ERR_UNSUPPORTED;
  if (N == 0) return SBW_OK;
  if (green_counts == nullptr || z == nullptr || (L > 0 && tokens == nullptr))
    return SBW_ERR_INVALID_ARG;
  if (row_stride > 0 && N > INT64_MAX / 4 / row_stride) return SBW_ERR_UNSUPPORTED;
  s = check_device();
  if (s != SBW_OK) return s;

  const uint64_t T = threshold_of(gamma);  // in [1, 2^32 - 1] for 0 < gamma < 1
  const uint32_t tm1 = static_cast<uint32_t>(T - 1);
  const int w = static_cast<int>(width);
  const DetectIO io{lengths, green_counts, scored, z};
  const bool ctx = seeding == SBW_SEED_CONTEXT;
  if (unique) {
    // a power of two, four times the scored positions where it fits, at least twice
    uint32_t slots = 64u;
    while (slots < 4 * positions && slots < kMaxUniqueSlots) slots *= 2u;
    if (w == 1) {
      if (ctx) launch_detect_unique<kContext, 1>(N, st, tokens, L, row_stride, w, key, tm1, gamma, slots, io);
      else launch_detect_unique<kSelfSalt, 1>(N, st, tokens, L, row_stride, w, key, tm1, gamma, slots, io);
    } else if (w <= kMidWidth) {
      if (ctx) launch_detect_unique<kContext, kMidWidth>(N, st, tokens, L, row_stride, w, key, tm1, gamma, slots, io);
      else launch_detect_unique<kSelfSalt, kMidWidth>(N, st, tokens, L, row_stride, w, key, tm1, gamma, slots, io);
    } else {
      if (ctx) launch_detect_unique<kContext, kMaxWidth>(N, st, tokens, L, row_stride, w, key, tm1, gamma, slots, io);
      else launch_detect_unique<kSelfSalt, kMaxWidth>(N, st, tokens, L, row_stride, w, key, tm1, gamma, slots, io);
    }
    return after_launch();
  }
  if (w == 1) {
    if (ctx) launch_detect<kContext, 1>(positions, st, tokens, N, L, row_stride, w, key, tm1, gamma, io);
    else launch_detect<kSelfSalt, 1>(positions, st, tokens, N, L, row_stride, w, key, tm1, gamma, io);
  } else if (w <= kMidWidth) {
    if (ctx) launch_detect<kContext, kMidWidth>(positions, st, tokens, N, L, row_stride, w, key, tm1, gamma, io);
    else launch_detect<kSelfSalt, kMidWidth>(positions, st, tokens, N, L, row_stride, w, key, tm1, gamma, io);
  } else {
    if (ctx) launch_detect<kContext, kMaxWidth>(positions, st, tokens, N, L, row_stride, w, key, tm1, gamma, io);
    else launch_detect<kSelfSalt, kMaxWidth>(positions, st, tokens, N, L, row_stride, w, key, tm1, gamma, io);
  }
  return after_launch();
}

// Token ids are 32-bit: a row holds fewer than 2^32 columns (its length is a 32-bit
// count), and a shard's last id, v_offset + V - 1, must fit.  v_offset >= 0.
constexpr int64_t kMaxTokenIds = int64_t{1} << 32;
bool ids_fit(int64_t V, int64_t v_offset) {
  return V < kMaxTokenIds && v_offset <= kMaxTokenIds - V;
}

// ---------------------------------------------------------------------------
// Scratch of sbw_watermark_argmax_noalloc: the per-segment partials that the other
// decoding calls keep in the caller's workspace, in an array of the code object, one
// copy per device, shared by every call on that device.  In host code the name is
// only a handle: the array's device address comes from hipGetSymbolAddress, resolved
// once per device with that device current, and only that address reaches a kernel.
// ---------------------------------------------------------------------------
constexpr int64_t kScratchElems = int64_t{1} << 18;  // uint64 partials: 2 MiB
static_assert(kScratchElems == SBW_NOALLOC_SCRATCH_ELEMS, "the header states the limit");
constexpr int kMaxDevices = 64;
std::atomic<uint64_t*> g_scratch_of_device[kMaxDevices];

}  // namespace
}  // namespace sbw

static __device__ __align__(256) uint64_t scratch[sbw::kScratchElems];

namespace sbw {
namespace {

// The device address of `scratch` on the current device (resolved on the first call
// made on that device).
sbw_status_t scratch_address(uint64_t** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) {
    g_last_hip_error = e;
    (void)hipGetLastError();
    return SBW_ERR_NO_DEVICE;
  }
  if (dev < 0 || dev >= kMaxDevices) return SBW_ERR_UNSUPPORTED;
  uint64_t* p = g_scratch_of_device[dev].load(std::memory_order_acquire);
  if (p == nullptr) {
    void* addr = nullptr;
    e = hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || addr == nullptr) {
      g_last_hip_error = e != hipSuccess ? e : hipErrorInvalidSymbol;
      (void)hipGetLastError();
      return SBW_ERR_HIP;
    }
    p = static_cast<uint64_t*>(addr);
    // every thread that resolves it gets the same address, so a race only repeats work
    g_scratch_of_device[dev].store(p, std::memory_order_release);
  }
  *out = p;
  return SBW_OK;
}

// Greedy decoding and sampling: validation, then the segment pass and the read-out.
// With use_scratch the partials go to the device's `scratch` array instead of
// `workspace` (which may then be null).
template <bool kSample>
sbw_status_t decode_impl(const void* logits, sbw_dtype_t dtype, int64_t B, int64_t V,
                         int64_t row_stride, const int32_t* context, int64_t width,
                         int64_t v_offset, uint64_t key, double gamma, float delta,
                         sbw_seeding_t seeding, const SampleArgs& sa, int32_t* tokens,
                         float* values, uint64_t* workspace, void* stream,
                         bool use_scratch = false) {
  if (B < 0 || V < 0 || row_stride < V || v_offset < 0) return SBW_ERR_INVALID_ARG;
  sbw_status_t s = check_width(width);
  if (s != SBW_OK) return s;
  if (dtype != SBW_F32 && dtype != SBW_BF16) return SBW_ERR_UNSUPPORTED;
  if (!valid_seeding(seeding)) return SBW_ERR_UNSUPPORTED;
  if (!(gamma >= 0.0 && gamma <= 1.0)) return SBW_ERR_GAMMA;
  if (!isfinite(delta)) return SBW_ERR_DELTA;
  if (!ids_fit(V, v_offset)) return SBW_ERR_UNSUPPORTED;
  if (B == 0) return SBW_OK;
  if (V == 0) return SBW_ERR_INVALID_ARG;  // no token to choose
  if (logits == nullptr || context == nullptr || tokens == nullptr ||
      (workspace == nullptr && !use_scratch))
    return SBW_ERR_INVALID_ARG;
  if (B > INT64_MAX / 4 / row_stride) return SBW_ERR_UNSUPPORTED;
  s = check_device();
  if (s != SBW_OK) return s;
  if (use_scratch) {
    s = scratch_address(&workspace);
    if (s != SBW_OK) return s;
  }

  // gamma == 0: nothing is green, every logit (and the value returned) is unchanged.
  const uint64_t T = threshold_of(gamma);
  const int none = T == 0 ? 1 : 0;
  const uint32_t tm1 = none ? 0u : static_cast<uint32_t>(T - 1);
  const float d = delta;
  const uint32_t vbase = static_cast<uint32_t>(v_offset);
  const uint32_t v32 = static_cast<uint32_t>(V);
  const int w = static_cast<int>(width);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (dtype == SBW_F32)
    dispatch_argmax<float, kSample>(logits, B, v32, row_stride, context, w, key, tm1, none, d, sa,
                                    seeding, vbase, tokens, values, workspace, st);
  else
    dispatch_argmax<uint16_t, kSample>(logits, B, v32, row_stride, context, w, key, tm1, none, d,
                                       sa, seeding, vbase, tokens, values, workspace, st);
  return after_launch();
}

}  // namespace
}  // namespace sbw

using namespace sbw;

extern "C" {

sbw_status_t sbw_watermark_shard(void* logits, sbw_dtype_t dtype, int64_t B, int64_t V,
                                 int64_t row_stride, const int32_t* context, int64_t width,
                                 int64_t v_offset, uint64_t key, double gamma, float delta,
                                 sbw_seeding_t seeding, void* stream) {
  if (B < 0 || V < 0 || row_stride < V || v_offset < 0) return SBW_ERR_INVALID_ARG;
  sbw_status_t s = check_width(width);
  if (s != SBW_OK) return s;
  if (dtype != SBW_F32 && dtype != SBW_BF16) return SBW_ERR_UNSUPPORTED;
  if (!valid_seeding(seeding)) return SBW_ERR_UNSUPPORTED;
  if (!(gamma >= 0.0 && gamma <= 1.0)) return SBW_ERR_GAMMA;
  if (!isfinite(delta)) return SBW_ERR_DELTA;
  if (!ids_fit(V, v_offset)) return SBW_ERR_UNSUPPORTED;  // token ids are 32-bit
  if (B == 0 || V == 0) return SBW_OK;
  if (logits == nullptr || context == nullptr) return SBW_ERR_INVALID_ARG;
  if (B > INT64_MAX / 4 / row_stride) return SBW_ERR_UNSUPPORTED;
  const uint64_t T = threshold_of(gamma);
  if (T == 0) return SBW_OK;  // nothing is green: the logits stay as they are
  s = check_device();
  if (s != SBW_OK) return s;

  const uint32_t vbase = static_cast<uint32_t>(v_offset);
  const uint32_t tm1 = static_cast<uint32_t>(T - 1);
  const uint32_t v32 = static_cast<uint32_t>(V);
  const int w = static_cast<int>(width);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (dtype == SBW_F32)
    dispatch_watermark<float>(logits, B, v32, row_stride, context, w, key, tm1, delta, seeding,
                              vbase, st);
  else
    dispatch_watermark<uint16_t>(logits, B, v32, row_stride, context, w, key, tm1, delta, seeding,
                                 vbase, st);
  return after_launch();
}

sbw_status_t sbw_watermark_window(void* logits, sbw_dtype_t dtype, int64_t B, int64_t V,
                                  int64_t row_stride, const int32_t* context, int64_t width,
                                  uint64_t key, double gamma, float delta, sbw_seeding_t seeding,
                                  void* stream) {
  return sbw_watermark_shard(logits, dtype, B, V, row_stride, context, width, 0, key, gamma, delta,
                             seeding, stream);
}

sbw_status_t sbw_watermark(void* logits, sbw_dtype_t dtype, int64_t B, int64_t V,
                           int64_t row_stride, const int32_t* prev_tokens, uint64_t key,
                           double gamma, float delta, sbw_seeding_t seeding, void* stream) {
  return sbw_watermark_window(logits, dtype, B, V, row_stride, prev_tokens, 1, key, gamma, delta,
                              seeding, stream);
}

sbw_status_t sbw_watermark_candidates(void* logits, sbw_dtype_t dtype, int64_t B, int64_t V,
                                      int64_t row_stride, const int32_t* candidates, int64_t k,
                                      const int32_t* context, int64_t width, uint64_t key,
                                      double gamma, float delta, sbw_seeding_t seeding,
                                      void* stream) {
  if (B < 0 || V < 0 || row_stride < V || k < 0) return SBW_ERR_INVALID_ARG;
  sbw_status_t s = check_width(width);
  if (s != SBW_OK) return s;
  if (dtype != SBW_F32 && dtype != SBW_BF16) return SBW_ERR_UNSUPPORTED;
  if (!valid_seeding(seeding)) return SBW_ERR_UNSUPPORTED;
  if (!(gamma >= 0.0 && gamma <= 1.0)) return SBW_ERR_GAMMA;
  if (!isfinite(delta)) return SBW_ERR_DELTA;
  if (V >= (int64_t{1} << 32) || k > kMaxCandidates) return SBW_ERR_UNSUPPORTED;
  if (B == 0 || V == 0 || k == 0) return SBW_OK;
  if (logits == nullptr || candidates == nullptr || context == nullptr) return SBW_ERR_INVALID_ARG;
  if (B > INT64_MAX / 4 / row_stride) return SBW_ERR_UNSUPPORTED;
  const uint64_t T = threshold_of(gamma);
  if (T == 0) return SBW_OK;  // nothing is green
  s = check_device();
  if (s != SBW_OK) return s;

  const uint32_t tm1 = static_cast<uint32_t>(T - 1);
  const uint32_t v32 = static_cast<uint32_t>(V);
  const int w = static_cast<int>(width);
  const int kk = static_cast<int>(k);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (dtype == SBW_F32)
    dispatch_candidates<float>(logits, B, v32, row_stride, candidates, kk, context, w, key, tm1,
                               delta, seeding, st);
  else
    dispatch_candidates<uint16_t>(logits, B, v32, row_stride, candidates, kk, context, w, key,
                                  tm1, delta, seeding, st);
  return after_launch();
}

sbw_status_t sbw_watermark_argmax(const void* logits, sbw_dtype_t dtype, int64_t B, int64_t V,
                                  int64_t row_stride, const int32_t* context, int64_t width,
                                  uint64_t key, double gamma, float delta, sbw_seeding_t seeding,
                                  int32_t* tokens, float* values, uint64_t* workspace,
                                  void* stream) {
  return decode_impl<false>(logits, dtype, B, V, row_stride, context, width, 0, key, gamma, delta,
                            seeding, SampleArgs{nullptr, 1.0f}, tokens, values, workspace, stream);
}

sbw_status_t sbw_watermark_argmax_shard(const void* logits, sbw_dtype_t dtype, int64_t B, int64_t V,
                                        int64_t row_stride, const int32_t* context, int64_t width,
                                        int64_t v_offset, uint64_t key, double gamma, float delta,
                                        sbw_seeding_t seeding, int32_t* tokens, float* values,
                                        uint64_t* workspace, void* stream) {
  return decode_impl<false>(logits, dtype, B, V, row_stride, context, width, v_offset, key, gamma,
                            delta, seeding, SampleArgs{nullptr, 1.0f}, tokens, values, workspace,
                            stream);
}

sbw_status_t sbw_watermark_sample(const void* logits, sbw_dtype_t dtype, int64_t B, int64_t V,
                                  int64_t row_stride, const int32_t* context, int64_t width,
                                  uint64_t key, double gamma, float delta, sbw_seeding_t seeding,
                                  const uint64_t* seeds, float inv_temperature, int32_t* tokens,
                                  float* scores, uint64_t* workspace, void* stream) {
  return sbw_watermark_sample_shard(logits, dtype, B, V, row_stride, context, width, 0, key, gamma,
                                    delta, seeding, seeds, inv_temperature, tokens, scores,
                                    workspace, stream);
}

sbw_status_t sbw_watermark_sample_shard(const void* logits, sbw_dtype_t dtype, int64_t B, int64_t V,
                                        int64_t row_stride, const int32_t* context, int64_t width,
                                        int64_t v_offset, uint64_t key, double gamma, float delta,
                                        sbw_seeding_t seeding, const uint64_t* seeds,
                                        float inv_temperature, int32_t* tokens, float* scores,
                                        uint64_t* workspace, void* stream) {
  if (!(isfinite(inv_temperature) && inv_temperature > 0.0f)) return SBW_ERR_INVALID_ARG;
  if (B > 0 && V > 0 && seeds == nullptr) return SBW_ERR_INVALID_ARG;
  return decode_impl<true>(logits, dtype, B, V, row_stride, context, width, v_offset, key, gamma,
                           delta, seeding, SampleArgs{seeds, inv_temperature}, tokens, scores,
                           workspace, stream);
}

sbw_status_t sbw_watermark_argmax_noalloc(const void* logits, sbw_dtype_t dtype, int64_t B,
                                          int64_t V, int64_t row_stride, const int32_t* context,
                                          int64_t width, uint64_t key, double gamma, float delta,
                                          sbw_seeding_t seeding, int32_t* tokens, float* values,
                                          void* stream) {
  // The partials must fit the static array: B * ceil(V / kArgmaxSegElems) elements,
  // compared by division so that no product overflows.
  if (B > 0 && V > 0 && B > kScratchElems / ((V + kArgmaxSegElems - 1) / kArgmaxSegElems))
    return SBW_ERR_UNSUPPORTED;
  return decode_impl<false>(logits, dtype, B, V, row_stride, context, width, 0, key, gamma, delta,
                            seeding, SampleArgs{nullptr, 1.0f}, tokens, values, nullptr, stream,
                            /*use_scratch=*/true);
}

int64_t sbw_watermark_argmax_workspace(int64_t B, int64_t V) {
  if (B <= 0 || V <= 0) return 0;
  return B * ((V + kArgmaxSegElems - 1) / kArgmaxSegElems);
}

sbw_status_t sbw_green_mask_window(uint32_t* bits, int64_t B, int64_t V, const int32_t* context,
                                   int64_t width, uint64_t key, double gamma,
                                   sbw_seeding_t seeding, void* stream) {
  if (B < 0 || V < 0) return SBW_ERR_INVALID_ARG;
  sbw_status_t s = check_width(width);
  if (s != SBW_OK) return s;
  if (!valid_seeding(seeding)) return SBW_ERR_UNSUPPORTED;
  if (!(gamma >= 0.0 && gamma <= 1.0)) return SBW_ERR_GAMMA;
  if (V >= (int64_t{1} << 32)) return SBW_ERR_UNSUPPORTED;
  if (B == 0 || V == 0) return SBW_OK;
  if (bits == nullptr || context == nullptr) return SBW_ERR_INVALID_ARG;
  const int64_t words = (V + 31) / 32;
  if (B > INT64_MAX / 4 / words) return SBW_ERR_UNSUPPORTED;
  s = check_device();
  if (s != SBW_OK) return s;

  const uint64_t T = threshold_of(gamma);
  const uint32_t tm1 = T == 0 ? 0u : static_cast<uint32_t>(T - 1);
  const int64_t num_words = B * words;
  const int64_t blocks = grid_for((num_words + kThreads - 1) / kThreads);
  const int w = static_cast<int>(width);
  const int none = T == 0 ? 1 : 0;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const uint32_t v32 = static_cast<uint32_t>(V), wpr = static_cast<uint32_t>(words);
  if (seeding == SBW_SEED_CONTEXT)
    hipLaunchKernelGGL((green_mask_kernel<kContext, kMaxWidth>), dim3(blocks), dim3(kThreads), 0,
                       st, bits, v32, wpr, context, w, key, tm1, none, num_words);
  else if (w == 1)
    hipLaunchKernelGGL((green_mask_kernel<kSelfSalt, 1>), dim3(blocks), dim3(kThreads), 0, st,
                       bits, v32, wpr, context, w, key, tm1, none, num_words);
  else
    hipLaunchKernelGGL((green_mask_kernel<kSelfSalt, kMaxWidth>), dim3(blocks), dim3(kThreads), 0,
                       st, bits, v32, wpr, context, w, key, tm1, none, num_words);
  return after_launch();
}

sbw_status_t sbw_green_mask(uint32_t* bits, int64_t B, int64_t V, const int32_t* prev_tokens,
                            uint64_t key, double gamma, sbw_seeding_t seeding, void* stream) {
  return sbw_green_mask_window(bits, B, V, prev_tokens, 1, key, gamma, seeding, stream);
}

sbw_status_t sbw_detect_window(const int32_t* tokens, int64_t N, int64_t L, int64_t row_stride,
                               int64_t width, uint64_t key, double gamma, sbw_seeding_t seeding,
                               int32_t* green_counts, double* z, void* stream) {
  return detect_impl(tokens, N, L, row_stride, nullptr, width, key, gamma, seeding, 0u,
                     green_counts, nullptr, z, static_cast<hipStream_t>(stream));
}

sbw_status_t sbw_detect_ex(const int32_t* tokens, int64_t N, int64_t L, int64_t row_stride,
                           const int32_t* lengths, int64_t width, uint64_t key, double gamma,
                           sbw_seeding_t seeding, uint32_t flags, int32_t* green_counts,
                           int32_t* scored, double* z, void* stream) {
  return detect_impl(tokens, N, L, row_stride, lengths, width, key, gamma, seeding, flags,
                     green_counts, scored, z, static_cast<hipStream_t>(stream));
}

sbw_status_t sbw_detect(const int32_t* tokens, int64_t N, int64_t L, int64_t row_stride,
                        uint64_t key, double gamma, sbw_seeding_t seeding,
                        int32_t* green_counts, double* z, void* stream) {
  return sbw_detect_window(tokens, N, L, row_stride, 1, key, gamma, seeding, green_counts, z,
                           stream);
}

const char* sbw_strerror(sbw_status_t status) {
  switch (status) {
    case SBW_OK: return "success";
    case SBW_ERR_INVALID_ARG: return "invalid argument (null pointer, negative size or stride too small)";
    case SBW_ERR_GAMMA: return "gamma out of range";
    case SBW_ERR_DELTA: return "delta is not finite";
    case SBW_ERR_UNSUPPORTED: return "unsupported dtype, seeding, width or size";
    case SBW_ERR_NO_DEVICE: return "no HIP device available";
    case SBW_ERR_HIP: return "HIP runtime or launch error";
  }
  return "unknown status";
}

const char* sbw_last_hip_error(void) { return hipGetErrorName(g_last_hip_error); }

const char* sbw_version(void) { return "0.5.0"; }

}  // extern "C"
