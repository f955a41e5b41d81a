// Device kernels of the PGC step for gfx950 (CDNA4, wave64).
//
// Gradient of the linear models (Sec. III; per-partition mean, Sec. IV-A /
// V-B evaluate one partition per worker per step).  Bound by HBM: every
// evaluated row is read exactly once, at 1 flop per byte.
//   * A row is spread over LANES x WAVES lanes, VEC chunks of 4 floats each,
//     so w and the gradient accumulators stay in registers for the whole
//     block.  Rows narrower than a wave share it: 64 / LANES rows per load, so
//     that a load still covers 1 KiB of consecutive rows.
//   * A chunk is a 16-byte load at any 4-byte alignment: rows of any length
//     and base address go at the rate of aligned ones.  The last chunk of a
//     row whose length is no multiple of 4 is read from the row's last four
//     floats, and the floats another lane owns are dropped from it.
//   * ROWS rows per lane are loaded per iteration (all loads, labels included,
//     issued before use), their dot products reduced by lane moves and, when a
//     row spans several waves, through a double-buffered LDS exchange (one
//     barrier per iteration);
//   * the loss slope scales the row still held in registers (axpy).  An
//     accumulator takes dump_rows rows, then moves to the lane's own sums in
//     LDS, so that rounding does not grow with the rows of a block;
//   * the rows sharing a wave and the GROUPS row groups of a block fold their
//     sums in a fixed order, so one partial per block leaves the kernel.  Rows of
//     4 to 128 features, of which an iteration of a block takes 64 to 2,048, fold
//     in 64 bits from the lane's sums on: in 32 bits the error of short runs is up
//     to twice that of sums of 16 rows;
//   * the evaluated rows of all partitions are cut into equal runs, one per
//     block, whatever the number of partitions: a block whose run crosses into
//     the next partition writes a partial for each.
// All reductions have a fixed order: results are bitwise reproducible.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "pgc_kernels.h"
#include "pgc_lanes.h"

namespace pgc {
namespace {

// VW floats per lane and load.  4: one 16-byte load, of which the hardware asks
// 4-byte alignment only; 1: rows of fewer than 4 features.
template <int VW> struct VecOf;
template <> struct VecOf<4> {
  typedef float T __attribute__((ext_vector_type(4)));
  typedef float Mem __attribute__((ext_vector_type(4), aligned(4)));
};
template <> struct VecOf<1> {
  typedef float T __attribute__((ext_vector_type(1)));
  typedef float Mem __attribute__((ext_vector_type(1)));
};

template <int VW>
__device__ __forceinline__ typename VecOf<VW>::T stream_load(const float* p) {
  // X is streamed once per step: non-temporal loads keep it from evicting
  // the small, reused vectors (w, partials) from the caches.
  return __builtin_nontemporal_load(reinterpret_cast<const typename VecOf<VW>::Mem*>(p));
}

template <int VW>
__device__ __forceinline__ typename VecOf<VW>::T plain_load(const float* p) {
  return *reinterpret_cast<const typename VecOf<VW>::Mem*>(p);
}

template <int VW>
__device__ __forceinline__ void plain_store(float* p, typename VecOf<VW>::T v) {
  *reinterpret_cast<typename VecOf<VW>::Mem*>(p) = v;
}

template <int VW>
__device__ __forceinline__ float hsum(typename VecOf<VW>::T v) {
  if constexpr (VW == 4) return (v[0] + v[1]) + (v[2] + v[3]);
  else return v[0];
}

template <int MODEL>
__device__ __forceinline__ float loss_slope(float z, float y) {
  if constexpr (MODEL == PGC_LOGISTIC) {
    return 1.0f / (1.0f + expf(-z)) - y;   // d/dz [log(1 + e^z) - y z]
  } else {
    return z - y;                          // d/dz [(z - y)^2 / 2]
  }
}

// Rows an accumulator sums before it moves to the lane's sums in LDS: 16, or 8 for
// the longest rows, whose runs hold few; d = 4,096 loses 0.5% to 8.
constexpr int dump_rows(int waves) { return waves == 16 ? 8 : 16; }
// Whether the accumulator starts again from what rounding took from the sum it moved to
// (two-sum, Knuth), so that the moves add nothing to the error: for the longest rows, whose
// blocks sum some 60 rows where sums of 16 would do for the fold in 64 bits (d = 20,000 in
// 16 x 1,000 rows: error 6.3e-8, without 8.1e-8, of sums of 16 rows 7.6e-8; times within 1%).
constexpr bool carry_rounding(int waves) { return waves == 16; }
// Whether a row's sums fold in 64 bits (rows of 4 to 128 features).
constexpr bool fold_wide(int vw, int lanes, int vec) { return vw == 4 && lanes < 64 && vec <= 2; }

template <int MODEL, int VW, int LANES, int WAVES, int VEC, int GROUPS, int ROWS>
__global__ __launch_bounds__(64 * WAVES * GROUPS)
void linear_gradient_kernel(LinearGradArgs a) {
  using V = typename VecOf<VW>::T;
  static_assert(LANES == 64 || WAVES == 1, "a row spans several waves only when it fills them");
  constexpr int kRowLanes = LANES * WAVES;
  constexpr int kGroupThreads = 64 * WAVES;
  constexpr int kSubs = 64 / LANES;             // rows side by side in a wave
  constexpr int kStep = GROUPS * ROWS * kSubs;  // rows per block and iteration
  const int lane = threadIdx.x % 64;
  const int wave = threadIdx.x / 64 % WAVES;
  const int group = threadIdx.x / kGroupThreads;
  const int sub = lane / LANES;
  const int row_lane = wave * LANES + lane % LANES;
  const int d = a.d;

  // A lane's chunk v is columns col(v) .. col(v) + VW - 1.  Only the last one
  // can lie past the row (own false: never loaded) or cross its end (keep < VW:
  // the lane's last `keep` floats are its own).  Two waves take a run of the row each,
  // which they read from end to end: VEC - 1 chunks per lane and half of the rest, in whole
  // cache lines.  Chunk by chunk in turn 4,096 features lose 0.5% at 4 GiB (592 us for 589)
  // and 1.7% at 100 MiB; 3,584 and 4,040 gain 1% at 1 GiB.  More waves gain nothing from
  // runs, and 16 lose up to 5%.
  constexpr bool kRuns = WAVES == 2;
  int first = row_lane * VW, end = d;
  if constexpr (kRuns) {
    const int rest = (d + VW - 1) / VW - 2 * (VEC - 1) * 64;   // 1 .. 128 chunks
    const int split = ((VEC - 1) * 64 + min((rest + 15) / 16 * 8, rest - 1)) * VW;
    first = lane * VW + (wave == 0 ? 0 : split);
    if (wave == 0) end = split;
  }
  constexpr int kNext = (kRuns ? LANES : kRowLanes) * VW;   // columns to the lane's next chunk
  const int last = first + (VEC - 1) * kNext;
  const bool own = last < end;
  const int keep = own ? min(d - last, VW) : VW;   // runs end with whole chunks but for the row's
  const int last_col = own ? last - (VW - keep) : 0;
  auto col = [&](int v) { return v == VEC - 1 ? last_col : first + v * kNext; };
  auto owned = [&](int v) { return v < VEC - 1 || own; };
  auto drop = [&](V x) {
#pragma unroll
    for (int i = 0; i + 1 < VW; ++i) x[i] = keep >= VW - i ? x[i] : 0.0f;
    return x;
  };

  // The accumulators of a chunk: an iteration's rows take turns, at most four each, and
  // their sums join in 64 bits.
  constexpr bool kWide = fold_wide(VW, LANES, VEC);
  constexpr bool kCarry = carry_rounding(WAVES);
  constexpr int kAccs = kWide && ROWS > 4 ? ROWS / 4 : 1;
  V wv[VEC], acc[kAccs][VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) wv[v] = owned(v) ? plain_load<VW>(a.w + col(v)) : V{};
  wv[VEC - 1] = drop(wv[VEC - 1]);

  __shared__ float dots[2][GROUPS][ROWS][WAVES];
  __shared__ V sums[VEC][kGroupThreads * GROUPS];
  __shared__ double wide[kWide ? GROUPS : 1][VEC][kWide ? 64 : 1];   // the row groups' folded sums
  int buf = 0;

  // The block's run of the evaluated rows, counted through the partitions.
  int64_t at = uniform(linear_block_row(a.rows, a.blocks, blockIdx.x));
  const int64_t run_end = uniform(linear_block_row(a.rows, a.blocks, blockIdx.x + int64_t{1}));
  for (int64_t e = uniform(short_div(at, a.m)); at < run_end; ++e) {
    const int64_t seg_end = min(run_end, (e + 1) * a.m);
    const int64_t skip = (e * a.part_stride + a.part_offset - e) * a.m;   // rows not evaluated before these
    const int64_t row_begin = at + skip, row_end = seg_end + skip;
    // Sums in LDS, rows in the accumulators.  With kCarry the rows move after their
    // iterations, not before the next (registers are few): LDS starts from zero and always
    // holds the sums, and what no rows follow stays (with 8 chunks it moves as well, for
    // which the test would spill).
    bool dumped = kCarry, held = false;
    auto dump = [&] {
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
#pragma unroll
        for (int t = 1; t < kAccs; ++t) {
          acc[0][v] += acc[t][v];
          acc[t][v] = V{};
        }
        if constexpr (kCarry) {
          const V old = sums[v][threadIdx.x], now = old + acc[0][v], part = now - old;
          const V lost = (old - (now - part)) + (acc[0][v] - part);
          sums[v][threadIdx.x] = now;
#pragma unroll
          for (int i = 0; i < VW; ++i) acc[0][v][i] = __builtin_isfinite(now[i]) ? lost[i] : 0.0f;
          __builtin_amdgcn_sched_barrier(0);   // registers are few: one chunk after the other
        } else {
          if (dumped) acc[0][v] += sums[v][threadIdx.x];
          sums[v][threadIdx.x] = acc[0][v];
          acc[0][v] = V{};
        }
      }
      dumped = true;
    };
    auto iterate = [&](int64_t base, auto ragged) {
      constexpr bool kRagged = decltype(ragged)::value;   // rows past row_end: read as zeros
      const int64_t r0 = base + group * (ROWS * kSubs) + sub;
      V x[ROWS][VEC];
      float label[ROWS];
#pragma unroll
      for (int r = 0; r < ROWS; ++r) {
        const int64_t row = r0 + r * kSubs;
        const bool in = !kRagged || row < row_end;
        const float* p = a.X + row * d;
#pragma unroll
        for (int v = 0; v < VEC; ++v) x[r][v] = (in && owned(v)) ? stream_load<VW>(p + col(v)) : V{};
        label[r] = in ? a.y[row] : 0.0f;
      }
      float dot[ROWS];
#pragma unroll
      for (int r = 0; r < ROWS; ++r) {
        x[r][VEC - 1] = drop(x[r][VEC - 1]);
        V p = x[r][0] * wv[0];
#pragma unroll
        for (int v = 1; v < VEC; ++v) p += x[r][v] * wv[v];
        dot[r] = lane_group_sum<LANES>(hsum<VW>(p));
      }
      if constexpr (WAVES > 1) {
        if (lane == 0) {
#pragma unroll
          for (int r = 0; r < ROWS; ++r) dots[buf][group][r][wave] = dot[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
          float s = dots[buf][group][r][0];
#pragma unroll
          for (int q = 1; q < WAVES; ++q) s += dots[buf][group][r][q];
          dot[r] = s;
        }
        buf ^= 1;
      }
#pragma unroll
      for (int r = 0; r < ROWS; ++r) {
        const float slope = (!kRagged || r0 + r * kSubs < row_end) ? loss_slope<MODEL>(dot[r], label[r]) : 0.0f;
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[r % kAccs][v] += slope * x[r][v];
      }
    };

#pragma unroll
    for (int t = 0; t < kAccs; ++t)
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[t][v] = V{};
    if constexpr (kCarry) {
#pragma unroll
      for (int v = 0; v < VEC; ++v) sums[v][threadIdx.x] = V{};
    }
    // Whole iterations, from a place in the run of the block's own (see
    // linear_spread_starts) round to it again; then the remainder.
    const int64_t whole = (row_end - row_begin) / kStep;   // kStep is a power of two
    const int64_t whole_end = row_begin + whole * kStep;
    int64_t start = row_begin;
    if (a.spread && whole > 1) {
      uint32_t h = blockIdx.x * 2654435761u;
      h = (h ^ (h >> 15)) * 0x85EBCA6Bu;
      start += uniform((h ^ (h >> 13)) % static_cast<uint32_t>(whole)) * kStep;
    }
    int64_t base = start, end = whole_end;
    for (int lap = 0; lap < 2; ++lap, base = row_begin, end = start) {
      while (base < end) {
        if (!kCarry && held) dump();
        for (int i = 0; i < dump_rows(WAVES) / ROWS && base < end; ++i, base += kStep) iterate(base, std::false_type{});
        if constexpr (!kCarry) held = true;
        else if (VEC == 8 || base < end || (lap == 0 && start > row_begin) || whole_end < row_end) dump();
      }
    }
    if (whole_end < row_end) {
      if (!kCarry && held) dump();
      iterate(whole_end, std::true_type{});
    }
    // The lane's sums, then the wave's side-by-side rows and the row groups fold.
    const int64_t slot = (blockIdx.x + (a.aligned ? 0 : e)) * static_cast<int64_t>(d);
    if constexpr (kWide) {
      // Lanes 16 i .. 16 i + 15 end with float i of the chunks.
      typedef double W __attribute__((ext_vector_type(VW)));
      const int i = lane / 16;
      double total[VEC];
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        W t = __builtin_convertvector(acc[0][v], W);
#pragma unroll
        for (int u = 1; u < kAccs; ++u) t += __builtin_convertvector(acc[u][v], W);
        if (dumped) t += __builtin_convertvector(sums[v][threadIdx.x], W);
        total[v] = lane_stride_sums<LANES>(t);
        if (group > 0) wide[group][v][lane] = total[v];
      }
      __syncthreads();
      if (group == 0 && lane % 16 < LANES) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
#pragma unroll
          for (int g = 1; g < GROUPS; ++g) total[v] += wide[g][v][lane];
          if (v < VEC - 1 || (own && keep >= VW - i)) {
            const int64_t at = slot + col(v) + i;
            if (a.wide) static_cast<double*>(a.partials)[at] = total[v];
            else static_cast<float*>(a.partials)[at] = static_cast<float>(total[v]);
          }
        }
      }
    } else {
      if (kCarry || dumped) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[0][v] += sums[v][threadIdx.x];
      }
#pragma unroll
      for (int off = LANES; off < 64; off <<= 1)
#pragma unroll
        for (int v = 0; v < VEC; ++v)
#pragma unroll
          for (int i = 0; i < VW; ++i) acc[0][v][i] += __shfl_xor(acc[0][v][i], off, 64);
      if constexpr (GROUPS > 1) {
        if (group > 0 && sub == 0) {
#pragma unroll
          for (int v = 0; v < VEC; ++v) sums[v][threadIdx.x] = acc[0][v];
        }
        __syncthreads();
        if (group == 0) {
#pragma unroll
          for (int v = 0; v < VEC; ++v)
#pragma unroll
            for (int g = 1; g < GROUPS; ++g) acc[0][v] += sums[v][g * kGroupThreads + threadIdx.x];
        }
      }
      if (group == 0 && sub == 0) {
        float* out = static_cast<float*>(a.partials) + slot;
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
          if (v < VEC - 1 || (own && keep == VW)) {
            plain_store<VW>(out + col(v), acc[0][v]);
          } else if (own) {
#pragma unroll
            for (int i = 1; i < VW; ++i)
              if (keep >= VW - i) out[last_col + i] = acc[0][v][i];
          }
        }
      }
    }
    at = seg_end;
    if (GROUPS > 1 && at < run_end) __syncthreads();   // group 0 has read every group's sums
  }
}

// Launch shapes by the row's 16-byte chunks: lanes and waves of a row, chunks
// per lane, row groups per block, rows per lane and iteration, and the blocks a
// launch aims for.  What bounds every class is the HBM stream, which asks for
// some 100 KiB of loads in flight per CU: a lane issues about 8 chunks before it
// waits for the first (chunks of one row, or of several short ones), 8 to 16
// waves per CU do so, and the lanes of a row grow by powers of two so that few
// idle.  All of a launch's blocks fit the chip at once and end together: 3 of 4
// waves per CU (4 where up to half of the lanes idle, 2 where nearly all carry 4
// chunks or more), or 1 of 8 or 16 waves for longer rows, of which a block has
// too few to balance otherwise.
// Chosen over 48 MiB to 3 GiB in 8 to 100 partitions, among 243 shapes on 256 to
// 1,024 blocks; each is within 5% of the best on average.  Kernel time for 1 GiB
// on MI355X (in brackets with a whole wave or more per row, scalar loads unless
// d % 4 == 0, and equal blocks per partition instead of equal blocks):
//   d = 20: 176 us (1,631); 69: 175 (503); 100: 170 (372); 200: 157 (218);
//   300: 154 (253); 512: 160 (179); 784: 155 (172); 1,001: 164 (264);
//   1,024: 151 (160, 194 in 12 partitions); 1,500: 155 (179); 2,048: 152 (163);
//   3,072: 154 (162); 4,096: 155 (154); 6,000: 155 (235); 8,192: 157 (192);
//   12,000: 162 (230); 16,384: 166 (194); 20,000: 165 (216); 32,768: 167 (184).
struct Shape { int max_chunks, lanes, waves, vec, groups, rows, blocks; };
constexpr Shape kShapes4[] = {
    {1, 1, 1, 1, 4, 8, 768},      {2, 2, 1, 1, 4, 8, 768},      {4, 4, 1, 1, 4, 8, 768},
    {6, 8, 1, 1, 4, 8, 1024},     {8, 8, 1, 1, 4, 8, 768},      {12, 16, 1, 1, 4, 8, 1024},
    {16, 16, 1, 1, 4, 8, 768},    {32, 16, 1, 2, 4, 4, 768},    {48, 16, 1, 3, 4, 2, 768},
    {56, 16, 1, 4, 4, 2, 768},    {64, 16, 1, 4, 4, 1, 512},    {96, 32, 1, 3, 4, 2, 768},
    {112, 32, 1, 4, 4, 2, 768},   {128, 32, 1, 4, 4, 1, 512},   {192, 64, 1, 3, 4, 2, 768},
    {224, 64, 1, 4, 4, 2, 768},   {256, 64, 1, 4, 4, 1, 512},   {320, 64, 1, 5, 4, 1, 512},
    {384, 64, 1, 6, 4, 1, 512},   {512, 64, 2, 4, 2, 2, 512},   {640, 64, 2, 5, 4, 1, 512},
    {768, 64, 2, 6, 4, 2, 256},   {896, 64, 2, 7, 4, 2, 256},   {1024, 64, 2, 8, 4, 2, 256},
    {1280, 64, 4, 5, 2, 2, 256},  {1536, 64, 4, 6, 2, 2, 256},  {2048, 64, 8, 4, 2, 2, 256},
    {2560, 64, 8, 5, 2, 1, 256},  {3072, 64, 8, 6, 2, 1, 256},  {4096, 64, 16, 4, 1, 2, 256},
    {5120, 64, 16, 5, 1, 1, 256}, {6144, 64, 16, 6, 1, 1, 256}, {7168, 64, 16, 7, 1, 1, 256},
    {8192, 64, 16, 8, 1, 1, 256}};
constexpr int kNumShapes = sizeof(kShapes4) / sizeof(kShapes4[0]);
// Rows of 1 to 3 features: one float per lane, four lanes per row.
constexpr Shape kShape1 = {1, 4, 1, 1, 4, 8, 768};

using GradKernel = void (*)(LinearGradArgs);

template <int MODEL, int I>
GradKernel pick(int index) {
  if constexpr (I == kNumShapes) {
    return nullptr;
  } else {
    constexpr Shape s = kShapes4[I];
    if (index == I) return linear_gradient_kernel<MODEL, 4, s.lanes, s.waves, s.vec, s.groups, s.rows>;
    return pick<MODEL, I + 1>(index);
  }
}

template <int MODEL>
GradKernel kernel_for(int d, int index) {
  constexpr Shape s = kShape1;
  if (d < 4) return linear_gradient_kernel<MODEL, 1, s.lanes, s.waves, s.vec, s.groups, s.rows>;
  return pick<MODEL, 0>(index);
}

// Index into kShapes4 of the class of d (0 for the rows of kShape1), or -1.
int shape_index(int d) {
  const int chunks = (d + 3) / 4;
  for (int i = 0; i < kNumShapes; ++i)
    if (chunks <= kShapes4[i].max_chunks) return i;
  return -1;
}

const Shape& shape_of(int d) {
  const int i = shape_index(d);
  return d < 4 ? kShape1 : kShapes4[i < 0 ? kNumShapes - 1 : i];
}

}  // namespace

// Runs of equal length start an equal distance apart and are read in step, so at
// some distances most blocks ask the same memory channels at once: 512 runs of
// 516 KiB read at 3.9 TB/s, of 504 or 528 KiB at 6.0 (MI355X; one length in twenty
// loses a tenth or more).  Started at scattered places they read at 6.1 whatever
// the length, 0 to 3% below the best; but lengths of a multiple of 64 KiB never
// collide (2 MiB: 7.1 TB/s in step, 6.7 scattered).
bool linear_spread_starts(int64_t rows, int64_t blocks, int64_t d) {
  return rows % blocks != 0 || rows / blocks * d * 4 % 65536 != 0;
}

LinearGradShape linear_grad_shape(int d) {
  const Shape& s = shape_of(d);
  return {s.blocks, s.groups * s.rows * (64 / s.lanes), fold_wide(d < 4 ? 1 : 4, s.lanes, s.vec)};
}

bool linear_grad_supported(int d, bool aligned16) {
  return d <= (aligned16 && d % 4 == 0 ? PGC_MAX_LINEAR_D : PGC_MAX_LINEAR_D_UNALIGNED);
}

hipError_t launch_linear_gradient(const LinearGradArgs& a, hipStream_t stream) {
  const int i = shape_index(a.d);
  if (a.d < 1 || i < 0) return hipErrorInvalidValue;
  GradKernel k = nullptr;
  if (a.model == PGC_LOGISTIC) k = kernel_for<PGC_LOGISTIC>(a.d, i);
  else if (a.model == PGC_LSQ) k = kernel_for<PGC_LSQ>(a.d, i);
  if (k == nullptr) return hipErrorInvalidValue;
  const Shape& s = shape_of(a.d);
  hipLaunchKernelGGL(k, dim3(a.blocks), dim3(64 * s.waves * s.groups), 0, stream, a);
  return hipGetLastError();
}

}  // namespace pgc
