// Post-gradient kernels of the PGC step for gfx950: the linear models' fused
// partial reduction + ring write + encode + masked decode + update, and the
// encode + masked decode + update alone (used after the MLP gradient).
// Sec. IV-A (FR encode / decode), Sec. V-A (real coefficients), Sec. V-B (CR).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "pgc_kernels.h"

namespace pgc {
namespace {

// Encode, masked decode and update of 256 columns by a 256-thread block: a
// thread owns 4 consecutive columns (16-byte ring loads; slots are padded to
// ld, a multiple of 256, so a block never leaves its slot), the four waves split
// the coded words (j = wave, wave + 4, ...), each word is summed in fp64, and
// the waves' decode partials are added in wave order.  Bound by HBM.  With more
// bytes than the 256 MiB cache in front of it holds, ring and coded words are
// streamed past the caches (kStream): 64 x 4 slots and 64 words of 814,090 columns,
// 1.04 GB, take 180 us (5.8 TB/s) instead of 225; 497 MiB 91 instead of 109, 298 MiB 57
// instead of 59 to 63.  20 MB take 10.0 us streamed, 9.5 not, as part of the ring is
// still cached there.
constexpr int kCodeCols = 256;
constexpr int64_t kStreamBytes = int64_t{256} << 20;
typedef float f4v __attribute__((ext_vector_type(4)));

template <bool kStream>
__global__ __launch_bounds__(256)
void code_kernel(CodeArgs a) {
  __shared__ double part[4][kCodeCols];
  const int lane = threadIdx.x % 64, sub = threadIdx.x / 64;
  const int64_t col = static_cast<int64_t>(blockIdx.x) * kCodeCols + 4 * lane;
  double ghat[4] = {0.0, 0.0, 0.0, 0.0};
  for (int j = sub; j < a.n_coded; j += 4) {
    double word[4] = {0.0, 0.0, 0.0, 0.0};
    for (int o = 0; o < a.c; ++o) {
      const int64_t slot = a.fr ? static_cast<int64_t>(j) * a.c + o
                                : static_cast<int64_t>(o) * a.n + (j + o) % a.n;
      const f4v* src = reinterpret_cast<const f4v*>(a.ring + slot * a.ld + col);
      const f4v v = kStream ? __builtin_nontemporal_load(src) : *src;
      const double cf = a.coef ? a.coef[j * a.c + o] : 1.0;
#pragma unroll
      for (int i = 0; i < 4; ++i) word[i] += cf * static_cast<double>(v[i]);
    }
    f4v out;
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = static_cast<float>(word[i]);
    f4v* dst = reinterpret_cast<f4v*>(a.coded + static_cast<int64_t>(j) * a.ld + col);
    if (kStream) __builtin_nontemporal_store(out, dst);
    else *dst = out;
    if (a.a[j] != 0.0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) ghat[i] += a.a[j] * word[i];
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) part[sub][4 * lane + i] = ghat[i];
  __syncthreads();
  const int c = threadIdx.x;   // one column per thread for the result
  const int64_t gc = static_cast<int64_t>(blockIdx.x) * kCodeCols + c;
  if (gc < a.q) {
    const double g = ((part[0][c] + part[1][c]) + part[2][c]) + part[3][c];
    a.decoded[gc] = static_cast<float>(g);
    a.w[gc] = static_cast<float>(static_cast<double>(a.w[gc]) - a.lr * g);
  }
}

// Loads N entries `stride` apart, from the `count`-th on the last one again.
template <class T, int N>
__device__ __forceinline__ void load_up_to(T (&t)[N], const T* p, int count, int64_t stride) {
#pragma unroll
  for (int i = 0; i < N; ++i) t[i] = p[min(i, count - 1) * stride];
}
// Adds the first `count` of N entries to s, in order.
template <class T, int N>
__device__ __forceinline__ void add_up_to(double& s, const T (&t)[N], int count) {
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (i < count) s += static_cast<double>(t[i]);
}
template <int N, class T>
__device__ __forceinline__ void load_and_add(double& s, const T* p, int count, int64_t stride) {
  T t[N];
  load_up_to<T, N>(t, p, count, stride);
  add_up_to<T, N>(s, t, count);
}

template <int N, class T>
__device__ __forceinline__ void load_and_add_all(double& s, const T* p, int64_t stride) {
  T t[N];
#pragma unroll
  for (int i = 0; i < N; ++i) t[i] = p[i * stride];
  add_up_to<T, N>(s, t, N);
}

// Sum in 64 bits and in order of `count` entries `stride` apart, with several loads in
// flight.  kUniform: the count is the same for all lanes, and a remainder takes fewer than
// two loads per entry; else the branches for that cost more than the loads.
template <bool kUniform, class T>
__device__ __forceinline__ double strided_sum(const T* p, int count, int64_t stride) {
  double s = 0.0;
  int b = 0;
  for (; b + 32 <= count; b += 32) load_and_add_all<32>(s, p + b * stride, stride);
  for (; b + 8 <= count; b += 8) load_and_add_all<8>(s, p + b * stride, stride);
  p += b * stride;
  count -= b;
  if (count > 4 || (!kUniform && count > 0)) load_and_add<7>(s, p, count, stride);
  else if (count > 2) load_and_add<4>(s, p, count, stride);
  else if (count > 0) load_and_add<2>(s, p, count, stride);
  return s;
}

// Block b owns columns [16 b, 16 b + 16).  It first folds every evaluated
// partition's block partials for those columns into the ring (fp64, block
// order, one (partition, column) pair per thread and round; bound by a memory
// latency and the index arithmetic of each round), then -- after a barrier, so
// the fresh slots written by its own threads are visible -- encodes, decodes
// and updates the same columns with the 16 lanes of each column splitting the
// coded words.  No block depends on another.
constexpr int kFusedCols = 16;
constexpr int kFusedSubs = 256 / kFusedCols;

template <class Partial>
__global__ __launch_bounds__(256)
void reduce_code_kernel(ReduceCodeArgs a) {
  __shared__ double part[kFusedSubs][kFusedCols];
  const CodeArgs& ca = a.code;
  const int64_t col0 = static_cast<int64_t>(blockIdx.x) * kFusedCols;
  const Partial* const partials = static_cast<const Partial*>(a.partials);
  const int pairs = a.n_eval * kFusedCols;
  auto there = [&](int pair) { return pair < pairs && col0 + pair % kFusedCols < ca.q; };
  auto put = [&](int pair, double s) {
    const float g = static_cast<float>(s * a.inv_m);
    const int64_t k = static_cast<int64_t>(pair / kFusedCols) * a.part_stride + a.part_offset;
    for (int pl = 0; pl < a.plane_count; ++pl)
      a.ring[((a.plane_first + pl) * static_cast<int64_t>(ca.n) + k) * ca.ld + col0 + pair % kFusedCols] = g;
  };
  // Up to 4 partials per partition, as many workers with few rows leave them: a thread loads
  // those of four pairs before it adds.  81 partitions of 16 rows of 371 features, one partial
  // each, take 8.5 us (10.5 pair by pair with seven loads each); 84 of 1,304, four each, 10.4
  // (11.9).
  auto few = [&](auto most) {
    constexpr int kMost = decltype(most)::value, kPairs = 4;
    for (int pair = threadIdx.x; pair < pairs; pair += 256 * kPairs) {
      Partial t[kPairs][kMost];
#pragma unroll
      for (int u = 0; u < kPairs; ++u) {
        const int at = pair + 256 * u;
        const int64_t first = static_cast<int64_t>(at / kFusedCols) * a.per_part;
        if (there(at)) load_up_to<Partial, kMost>(t[u], partials + first * ca.q + col0 + at % kFusedCols, a.per_part, ca.q);
      }
#pragma unroll
      for (int u = 0; u < kPairs; ++u) {
        if (!there(pair + 256 * u)) continue;
        double s = 0.0;
        add_up_to<Partial, kMost>(s, t[u], a.per_part);
        put(pair + 256 * u, s);
      }
    }
  };
  // range(e, &count): partition e's first partial.
  auto many = [&](auto uniform, auto range) {
    for (int pair = threadIdx.x; pair < pairs; pair += 256) {
      if (!there(pair)) continue;
      int count;
      const int64_t first = range(pair / kFusedCols, &count);
      put(pair, strided_sum<decltype(uniform)::value>(partials + first * ca.q + col0 + pair % kFusedCols, count, ca.q));
    }
  };
  if (a.per_part == 1) {
    few(std::integral_constant<int, 1>{});
  } else if (a.per_part == 2) {
    few(std::integral_constant<int, 2>{});
  } else if (a.per_part == 3 || a.per_part == 4) {
    few(std::integral_constant<int, 4>{});
  } else if (a.per_part > 0) {   // equal numbers stay in scalar registers: 5.0 us for 5.4, 64 each of 12
    many(std::true_type{}, [&](int e, int* count) {
      *count = a.per_part;
      return static_cast<int64_t>(e) * a.per_part;
    });
  } else {
    many(std::false_type{}, [&](int e, int* count) {
      const int64_t rows = a.m * a.n_eval, block = linear_row_block(rows, a.blocks, e * a.m);
      *count = static_cast<int>(linear_row_block(rows, a.blocks, (e + 1) * a.m - 1) - block) + 1;
      return block + e;
    });
  }
  __syncthreads();

  const int lane = threadIdx.x % kFusedCols, sub = threadIdx.x / kFusedCols;
  const int64_t col = col0 + lane;
  const bool live = col < ca.q;
  double ghat = 0.0;
  if (live) {
    for (int j = sub; j < ca.n_coded; j += kFusedSubs) {
      double word = 0.0;
      for (int o = 0; o < ca.c; ++o) {
        const int64_t slot = ca.fr ? static_cast<int64_t>(j) * ca.c + o
                                   : static_cast<int64_t>(o) * ca.n + (j + o) % ca.n;
        const double v = static_cast<double>(a.ring[slot * ca.ld + col]);
        word += ca.coef ? ca.coef[j * ca.c + o] * v : v;
      }
      ca.coded[static_cast<int64_t>(j) * ca.ld + col] = static_cast<float>(word);
      if (ca.a[j] != 0.0) ghat += ca.a[j] * word;
    }
  }
  part[sub][lane] = ghat;
  __syncthreads();
  if (sub == 0 && live) {
    double g = part[0][lane];
#pragma unroll
    for (int i = 1; i < kFusedSubs; ++i) g += part[i][lane];
    ca.decoded[col] = static_cast<float>(g);
    ca.w[col] = static_cast<float>(static_cast<double>(ca.w[col]) - ca.lr * g);
  }
}

}  // namespace

hipError_t launch_reduce_code(const ReduceCodeArgs& a, hipStream_t stream) {
  dim3 grid(static_cast<unsigned>((a.code.q + kFusedCols - 1) / kFusedCols));
  if (a.wide) hipLaunchKernelGGL(reduce_code_kernel<double>, grid, dim3(256), 0, stream, a);
  else hipLaunchKernelGGL(reduce_code_kernel<float>, grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_code(const CodeArgs& a, hipStream_t stream) {
  dim3 grid(static_cast<unsigned>((a.q + kCodeCols - 1) / kCodeCols));
  const int64_t bytes = (static_cast<int64_t>(a.n_coded) * a.c + a.n_coded) * a.ld * 4;
  if (bytes > kStreamBytes) hipLaunchKernelGGL(code_kernel<true>, grid, dim3(256), 0, stream, a);
  else hipLaunchKernelGGL(code_kernel<false>, grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace pgc
