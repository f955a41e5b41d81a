// Launchers of the PGC step's device kernels (gfx950).  Internal to the library.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "pgc.h"

namespace pgc {

// a / b for a >= 0, b > 0, in 32 bits where both fit: a 64-bit division takes a lane
// some 0.5 us, which the smallest steps notice.
__host__ __device__ inline int64_t short_div(int64_t a, int64_t b) {
  return ((a | b) >> 32) == 0 ? static_cast<int64_t>(static_cast<uint32_t>(a) / static_cast<uint32_t>(b)) : a / b;
}

// First of block b's rows when `blocks` blocks share `rows` rows (b = blocks: the
// end): floor(b * rows / blocks).
__host__ __device__ inline int64_t linear_block_row(int64_t rows, int64_t blocks, int64_t b) {
  const int64_t each = short_div(rows, blocks);
  return b * each + short_div(b * (rows - each * blocks), blocks);
}
// The block whose rows hold row r.
__host__ __device__ inline int64_t linear_row_block(int64_t rows, int64_t blocks, int64_t r) {
  return short_div((r + 1) * blocks - 1, rows);
}

// Per-partition gradient of a linear model (Sec. III with a mean over each
// partition's rows).  The rows of the evaluated partitions k = e * part_stride +
// part_offset, e < n_eval, are counted through, and each of `blocks` blocks takes
// an equal run of them.  For every partition that block b's run touches it sums
//   slope(x_r . w, y_r) * x_r
// over its rows there and writes the sum (fp64 when wide, else fp32) to
// partials[slot * d].  When the runs
// never cross a partition's end (aligned: n_eval divides blocks) slot = b, else
// slot = b + e, which grows by one or two from each sum to the next.
struct LinearGradArgs {
  const float* X;          // N x d row-major
  const float* y;          // N
  const float* w;          // d
  void* partials;          // (blocks + (aligned ? 0 : n_eval - 1)) * d
  int64_t m;               // rows per partition
  int64_t rows;            // n_eval * m
  int32_t d;
  int32_t blocks;          // at most rows
  int32_t aligned;
  int32_t wide;            // only where the shape folds in 64 bits
  int32_t spread;          // start each block at a scattered place in its run
  int32_t part_stride;
  int32_t part_offset;
  int32_t model;           // PGC_LOGISTIC or PGC_LSQ
};

// Whether the step takes d features: up to PGC_MAX_LINEAR_D when d % 4 == 0 and X
// and w are 16-byte aligned, else up to PGC_MAX_LINEAR_D_UNALIGNED.
bool linear_grad_supported(int d, bool aligned16);
// Blocks per launch that the gradient grid aims for, the rows a block takes at
// once, and whether it folds them in 64 bits (by d only, so the grid, and with it every result, is independent of pointer
// alignment and device).
struct LinearGradShape {
  int target_blocks;
  int rows_per_iteration;
  bool folds_wide;
};
LinearGradShape linear_grad_shape(int d);

// Whether the blocks' runs are better read from scattered starts.
bool linear_spread_starts(int64_t rows, int64_t blocks, int64_t d);

hipError_t launch_linear_gradient(const LinearGradArgs& a, hipStream_t s);

// Encode, masked decode and update, column by column:
//   coded_j = sum_o coef(j, o) * ring[slot(j, o)]          (Sec. IV-A, V-A, V-B)
//   ghat    = sum_j a_j * coded_j  over j with a_j != 0    (stragglers skipped)
//   w      <- w - lr * ghat
// FR (fr = 1): j is a group, slot(j, o) = plane 0, partition j*c + o.
// CR: j is a worker, slot(j, o) = plane o, partition (j + o) mod n.
// coef == nullptr means unit coefficients; else coef[j * c + o] (fp64).
struct CodeArgs {
  const float* ring;       // planes x n x ld  (ld >= q, a multiple of 256)
  float* coded;            // n_coded x ld
  float* decoded;          // q
  float* w;                // q
  const double* coef;      // n_coded x c, or nullptr
  int64_t q;
  int64_t ld;
  double lr;
  int32_t n;
  int32_t c;
  int32_t n_coded;
  int32_t fr;
  double a[PGC_MAX_N];     // decode weight per coded index (already scaled)
};
hipError_t launch_code(const CodeArgs& a, hipStream_t s);

// The linear models' block partials folded into the ring, then the code step,
// in one launch: for each evaluated e (partition k = e * part_stride +
// part_offset) and p < plane_count,
//   ring[(plane_first + p) * n + k][:] = inv_m * sum of e's partials
// (fp64, block order; the gradient kernel's slots), then encode / decode / update
// of the same columns.
struct ReduceCodeArgs {
  CodeArgs code;
  float* ring;             // the ring code.ring reads, written here first
  const void* partials;    // as LinearGradArgs::partials
  double inv_m;
  int64_t m;
  int32_t n_eval;
  int32_t blocks;
  int32_t per_part;        // partials of each e where the runs are aligned, else 0
  int32_t wide;            // fp64 partials
  int32_t part_stride;
  int32_t part_offset;
  int32_t plane_first;
  int32_t plane_count;
};
hipError_t launch_reduce_code(const ReduceCodeArgs& a, hipStream_t s);

// ---------------------------------------------------------------------------
// Two-layer MLP (d_in -> hidden, ReLU -> classes, softmax cross-entropy), bf16
// operands with fp32 accumulation on MFMA.  Parameters w (fp32) are laid out
// W1[d_in][hidden], b1[hidden], W2[hidden][classes], b2[classes].
// Shape limits: d_in % 8 == 0, hidden % 256 == 0 and <= 1024, classes <= 16.
// ---------------------------------------------------------------------------

constexpr int kMlpMaxClasses = 16;
constexpr int kMlpMaxHidden = 1024;

// bf16 copies of the weights for the GEMMs.  W1F: for each slice ks of 32
// features (kslices = ceil(d_in / 32), zero past d_in) and tile ht of 16 hidden
// units one MFMA fragment of 1 KiB, element (32 ks + 8 g + j, 16 ht + i) at
//   W1F[((ks * hidden / 16 + ht) * 64 + 16 g + i) * 8 + j];
// W2T[16][hidden] and W2p[hidden][16] (zero past `classes`).
struct MlpCastArgs {
  const float* w;
  __bf16* W1F;
  __bf16* W2T;
  __bf16* W2p;
  int32_t d_in, kslices, hidden, classes;
};
hipError_t launch_mlp_cast(const MlpCastArgs& a, hipStream_t s);

// dZ1 layout, blocked by 16 rows: element (r, h) of evaluated partition e at
// dZ1[((e * m_pad / 16 + r / 16) * hidden + h) * 16 + r % 16], r < m_pad (a
// multiple of 64; zero for r >= m).  A 16-row tile is one contiguous run, and
// 8 consecutive rows of one hidden unit are 16 contiguous bytes.
__host__ __device__ inline int64_t mlp_dz1_index(int64_t m_pad, int32_t hidden, int32_t e, int64_t r, int32_t h) {
  return ((static_cast<int64_t>(e) * (m_pad / 16) + r / 16) * hidden + h) * 16 + r % 16;
}

// For each evaluated partition k = e * part_stride + part_offset, e < n_eval:
// H = bf16(relu(X W1 + b1)) of its rows, logits, softmax, dZ2 = (p - onehot(y)) / m,
// and dZ1 = (dZ2 W2^T) masked by H > 0, written in the blocked layout above
// (rows m .. m_pad - 1 as zeros).  The partitions' tiles_per_part row tiles are
// counted through and `blocks` blocks take an equal part of them each, in `runs` equal
// runs; the sums over run r's rows (r < blocks * runs) of partition e go to
// partials[(r + e) * pstride]:
// dW2^T[16][hidden] in MFMA order (class 4 g + j of unit 16 ht + i at
// ((ht * 4 + g) * 16 + i) * 4 + j; classes past the last group of four unwritten),
// db1[hidden], db2[16].
struct MlpRowsArgs {
  const __bf16* X;
  const int32_t* y;
  const __bf16* W1F;
  const __bf16* W2T;
  const __bf16* W2p;
  const float* b1;
  const float* b2;
  __bf16* dZ1;
  float* partials;
  int64_t m, m_pad, pstride;
  float inv_m;
  int32_t d_in, kslices, classes, n_eval, blocks, runs, part_stride, part_offset;
};
struct MlpRowsGrid {
  int64_t tiles_per_part = 0;
  int32_t blocks = 0;
  int32_t runs = 1;    // of a block
  int shape = 0;
};
MlpRowsGrid mlp_rows_grid(int64_t m_pad, int32_t n_eval, int32_t kslices, int32_t hidden);
hipError_t launch_mlp_rows(const MlpRowsArgs& a, int32_t hidden, int shape, hipStream_t s);

// The rows kernel's sums, as MlpRowsArgs describes them.
struct MlpSmallParts {
  const float* partials;
  int64_t tiles_per_part, pstride;
  int32_t runs, classes;   // runs of all blocks
};

// dW1[i][h] = sum_r X[k*m + r][i] dZ1(e; r, h), written into the ring slot of
// partition k: ring[((plane * n + k) * ld) + i * hidden + h].  With splits > 1 a
// partition's rows are cut into that many equal runs of 64-row steps, whose sums go
// to split_sums[(e * splits + split) * d_in * hidden + ..]; launch_mlp_reduce folds
// them into the slots, and always writes the slots' b1, W2 and b2 parts from the rows
// kernel's sums (fp64, fixed order).
struct MlpWgradArgs {
  const __bf16* X;
  const __bf16* dZ1;
  float* ring;
  float* split_sums;
  MlpSmallParts small;
  int64_t m, m_pad, ld;
  int32_t d_in, hidden, n, plane, n_eval, splits, part_stride, part_offset;
};
int mlp_wgrad_splits(int64_t m_pad, int32_t n_eval, int32_t d_in, int32_t hidden);
hipError_t launch_mlp_wgrad(const MlpWgradArgs& a, hipStream_t s);
hipError_t launch_mlp_reduce(const MlpWgradArgs& a, hipStream_t s);

// Header of a saved pipeline state: the first kStateHeaderBytes bytes of the
// caller's buffer (the rest of the struct's space is zero), followed by the
// ring.  Every field but t must match the loading context.
struct StateHeader {
  uint64_t magic;     // kStateMagic
  uint64_t version;   // kStateVersion
  int64_t t, N, q, ld;
  uint64_t code_seed;
  int32_t scheme, n, c, model, d_in, hidden, classes, planes;
};
constexpr uint64_t kStateMagic = 0x4554415453434750ull;   // the bytes "PGCSTATE"
constexpr uint64_t kStateVersion = 1;
constexpr size_t kStateHeaderBytes = 256;
static_assert(sizeof(StateHeader) <= kStateHeaderBytes && sizeof(StateHeader) % 8 == 0, "state header");
// Writes h (zero-padded to kStateHeaderBytes) to out, which is 8-byte aligned.
hipError_t launch_write_state_header(const StateHeader& h, void* out, hipStream_t s);

}  // namespace pgc
