// Two-layer MLP gradient of the PGC step on gfx950: bf16 MFMA with fp32
// accumulation (the per-partition gradient of Sec. III for a network model;
// every worker evaluates one partition per step, Sec. IV-A / V-B).
//
// Per step, for the evaluated partitions:
//   cast     w (fp32) -> W1F, W2T, W2p (bf16 copies laid out for the MFMAs)
//   rows     H = relu(X W1 + b1), kept in registers     MFMA 16x16x32; then
//            logits = H W2 + b2, softmax, dZ2 = (p - onehot) / m,
//            dZ1 = (dZ2 W2^T) * [H > 0] (16-row blocked), and block
//            partials of dW2 = H^T dZ2, db1, db2         MFMA 16x16x16
//   wgrad    dW1 = X^T dZ1 straight into the ring slot  MFMA 16x16x32, both tiles
//            loaded straight into LDS, X fragments by transposing LDS reads; few
//            partitions split their rows over several blocks
//   reduce   rows partials -> b1, W2, b2 parts of the ring slot, and the sums of
//            the weight gradient's splits (fp64, fixed order)
//
// MFMA lane layouts (gfx950, wave64; l = lane, lr = l % 16, lg = l / 16):
//   16x16x32 bf16: A[lr][8 lg + j], B[8 lg + j][lr], j < 8;  D[4 lg + i][lr]
//   16x16x16 bf16: A[lr][4 lg + j], B[4 lg + j][lr], j < 4;  D[4 lg + i][lr]
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "pgc_kernels.h"
#include "pgc_lanes.h"

namespace pgc {
namespace {

typedef __bf16 bf16;
typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x4 mfma_k32(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_k16(bf16x4 a, bf16x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

template <class T>
__device__ __forceinline__ T load_vec(const bf16* p) { return *reinterpret_cast<const T*>(p); }

// ---------------------------------------------------------------------------
// cast: W1 and W2 in bf16, in the order in which the rows kernel reads them.
// One thread per 16 bytes of W1F (its loads are 64-byte pieces of W1's rows),
// then one per element of the two W2 tables.
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256)
void mlp_cast_kernel(MlpCastArgs a) {
  const int htiles = a.hidden / 16;
  const int64_t w1_items = static_cast<int64_t>(a.kslices) * htiles * 64;
  const int64_t id = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (id < w1_items) {
    const int lane = static_cast<int>(id % 64);
    const int64_t frag = id / 64;
    const int h = static_cast<int>(frag % htiles) * 16 + (lane & 15);
    const int64_t k0 = frag / htiles * 32 + (lane >> 4) * 8;
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = static_cast<bf16>(k0 + j < a.d_in ? a.w[(k0 + j) * a.hidden + h] : 0.0f);
    *reinterpret_cast<bf16x8*>(a.W1F + id * 8) = v;
    return;
  }
  const int64_t idx = id - w1_items;
  if (idx >= static_cast<int64_t>(a.hidden) * kMlpMaxClasses) return;
  const int h = static_cast<int>(idx / kMlpMaxClasses), c = static_cast<int>(idx % kMlpMaxClasses);
  const int64_t w2 = static_cast<int64_t>(a.d_in) * a.hidden + a.hidden;
  const float v = c < a.classes ? a.w[w2 + static_cast<int64_t>(h) * a.classes + c] : 0.0f;
  a.W2T[static_cast<int64_t>(c) * a.hidden + h] = static_cast<bf16>(v);
  a.W2p[idx] = static_cast<bf16>(v);
}

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void global_void;

// 16 bytes from global memory to LDS: lane l of the wave writes lds_wave_base + 16 l.
__device__ __forceinline__ void load_lds16(const void* src, void* lds_wave_base) {
  __builtin_amdgcn_global_load_lds((global_void*)src, (lds_void*)lds_wave_base, 16, 0, 0);
}

// 16 bytes from a wave-uniform base plus a per-lane byte offset to a wave-uniform LDS
// address, unknown to the compiler's wait insertion: before plain LDS reads
// that follow the builtin it waits for every outstanding load of this kind (it
// cannot tell the buffers apart), which would drain the prefetch.  The caller
// orders the loads with wait_vmcnt and barriers; the compiler's own counted waits
// only get stricter by loads that it does not count.  m0, which the load reads its LDS
// address from when it is issued, is the compiler's to use: it is put back.
__device__ __forceinline__ void load_lds16_async(const void* base, uint32_t offset_bytes, uint32_t lds_wave_base) {
  uint32_t m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b32 m0, %0"
               : "=&s"(m0) : "v"(offset_bytes), "s"(base), "s"(lds_wave_base) : "memory");
}

// Workgroup barrier that orders LDS only: the wave's own LDS reads and writes
// complete (lgkmcnt 0) before it, but outstanding global loads and stores do
// not have to, unlike the release fence of __syncthreads(), which would drain
// every prefetch.  Callers wait for the global loads they need with
// wait_vmcnt.  The empty asm statements keep the compiler from moving memory
// accesses across it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);   // vmcnt 63 (no wait), expcnt 7, lgkmcnt 0
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The wave's own LDS reads and writes complete.
__device__ __forceinline__ void lds_wait() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);
  asm volatile("" ::: "memory");
}

// Swizzle of the 16-byte chunks of an X stage's 128-byte rows: chunk ch of row r
// sits at slot ch ^ x_swizzle(r).  It depends on the row within its 16-row group,
// and the rows of a fragment read spread over the slots.
__device__ __forceinline__ int x_swizzle(int row) { return (row & 7) ^ ((row >> 3) & 1); }

// s_waitcnt with vmcnt = n (n < 16) and the other counters left alone.
template <int n>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(n >= 0 && n < 16, "vmcnt field");
  __builtin_amdgcn_s_waitcnt(0x0F70 | n);
}

constexpr int kXcds = 8;

typedef bf16 bf16x4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x4v lds_bf16x4;

__device__ __forceinline__ uint32_t lds_address(const bf16* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_bf16x4*)p));
}

// NT transposing 8-byte LDS reads, 32 bytes apart, and the wait for them.  One
// block of inline assembly: for the builtin the compiler waits for every
// outstanding direct-to-LDS load and store first (it cannot tell the buffers
// apart).  The memory clobber keeps it behind the LDS writes it reads.
template <int NT>
__device__ __forceinline__ void read_tr16(uint32_t addr, bf16x4v* v) {
  static_assert(NT == 2 || NT == 4 || NT == 6 || NT == 8, "reads");
  if constexpr (NT == 2) {
    asm volatile("ds_read_b64_tr_b16 %0, %2\n\tds_read_b64_tr_b16 %1, %2 offset:32\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]) : "v"(addr) : "memory");
  } else if constexpr (NT == 4) {
    asm volatile("ds_read_b64_tr_b16 %0, %4\n\tds_read_b64_tr_b16 %1, %4 offset:32\n\t"
                 "ds_read_b64_tr_b16 %2, %4 offset:64\n\tds_read_b64_tr_b16 %3, %4 offset:96\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]) : "v"(addr) : "memory");
  } else if constexpr (NT == 6) {
    asm volatile("ds_read_b64_tr_b16 %0, %6\n\tds_read_b64_tr_b16 %1, %6 offset:32\n\t"
                 "ds_read_b64_tr_b16 %2, %6 offset:64\n\tds_read_b64_tr_b16 %3, %6 offset:96\n\t"
                 "ds_read_b64_tr_b16 %4, %6 offset:128\n\tds_read_b64_tr_b16 %5, %6 offset:160\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5])
                 : "v"(addr) : "memory");
  } else {
    asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:32\n\t"
                 "ds_read_b64_tr_b16 %2, %8 offset:64\n\tds_read_b64_tr_b16 %3, %8 offset:96\n\t"
                 "ds_read_b64_tr_b16 %4, %8 offset:128\n\tds_read_b64_tr_b16 %5, %8 offset:160\n\t"
                 "ds_read_b64_tr_b16 %6, %8 offset:192\n\tds_read_b64_tr_b16 %7, %8 offset:224\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]),
                   "=&v"(v[7])
                 : "v"(addr) : "memory");
  }
}

// ---------------------------------------------------------------------------
// rows: forward, softmax and the backward pass down to dZ1 in one kernel, so
// that H never leaves the chip.  A block of 8 waves holds BM = 16 MT rows by
// all hidden units in accumulators (wave w: units 16 NT w ..), and walks an
// equal run of the evaluated partitions' row tiles.
//   H^T = relu(W1^T X^T + b1), K slices of 32 columns.
//     W1F comes from L2 in fragment order, each wave's fragments into a ring of
//     WB slices of its own in LDS: no barrier and no swizzle, the wave waits for
//     its own loads.  X rows, shared by the waves, go through two stages of two
//     slices (swizzled 128-byte rows), one barrier per stage: within it the waves
//     drift apart, and one's LDS reads run beside another's MFMAs.
//   logits^T = W2^T H^T: the MFMA result H^T is the next one's B operand as it
//     stands, so the logits come straight from registers.  The waves' partial
//     logits meet in LDS; wave w does the softmax of 16-row tiles w, w + 8, ..
//     and leaves dZ2 there, both ways round.
//   dH = dZ2 W2^T, masked by H > 0, is dZ1; dW2^T += dZ2^T H.  Both want H with
//     its rows in the registers: each wave turns its 16 x 16 NT tiles through its
//     own part of the ring (transposing LDS reads).
// The next tile's first slices are loaded while the softmax runs, and have
// landed before the first dZ1 store is issued, so no wait of the next tile
// includes the stores of this one before a whole slice has passed.
// Bound by the loads of W1F and by the slices' barriers: 1,048,576 rows of
// 784 -> 1024 -> 10 take 2.22 ms (0.67 ms of MFMAs; 1.51 ms without the loads),
// against 1.94 + 0.78 ms for a forward kernel that writes H and a head that reads it.
// ---------------------------------------------------------------------------

constexpr int kRowsThreads = 512, kRowsWaves = 8;

template <int NT, int MT, int WB>
__global__ __launch_bounds__(kRowsThreads, 1)
void mlp_rows_kernel(MlpRowsArgs a) {
  constexpr int kBM = 16 * MT, kHidden = 16 * NT * kRowsWaves;
  constexpr int kXStage = kBM * 64;                     // bf16: two K slices
  constexpr int kWSlice = NT * 512;                     // bf16 per wave
  constexpr int kXLoads = (MT + 3) / 4;                 // X loads per lane and stage (16 MT chunks per wave)
  constexpr int kTrLd = 16 * NT + 16;                   // row stride of the transposing area (bf16): the row
                                                        // pieces of a read hit distinct banks
  // Loads that may be outstanding when W1F's slice s is waited for.  After it came
  // W1F's slices up to s + WB - 2 and, at odd s, X's next stage; at even s that
  // stage is needed, and only one slice of W1F came after it.
  constexpr int kOddInFlight = (WB - 2) * NT + kXLoads, kEvenInFlight = WB > 2 ? NT : 0;
  static_assert(MT * 1024 <= (WB - 1) * kWSlice * 2 && 16 * kTrLd <= (WB - 1) * kWSlice,
                "the ring past its first slice holds the partial logits, then the transposing area");
  __shared__ __attribute__((aligned(16))) bf16 xs[2 * kXStage];
  __shared__ __attribute__((aligned(16))) bf16 ring[kRowsWaves * WB * kWSlice];
  __shared__ __attribute__((aligned(16))) bf16 dzs[MT][2][256];   // dZ2 [row][class], [class][row]
  __shared__ float db2s[kRowsWaves][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const int h0 = wave * 16 * NT;
  bf16* const mine = ring + wave * (WB * kWSlice);
  bf16* const area = mine + kWSlice;
  const uint32_t xs_at = lds_address(xs);
  const uint32_t mine_at = lds_address(ring) + static_cast<uint32_t>(wave * (WB * kWSlice * 2));

  const int64_t tiles_per_part = (a.m_pad + kBM - 1) / kBM;
  const int64_t tiles = tiles_per_part * a.n_eval;
  int64_t t = uniform(linear_block_row(tiles, a.blocks, blockIdx.x));
  const int64_t t_end = uniform(linear_block_row(tiles, a.blocks, blockIdx.x + int64_t{1}));
  const int kslices = a.kslices;
  const int dchunks = a.d_in / 8;

  // This lane's chunks of every X stage: row xrow + 8 u of the tile, slot
  // lane % 8, which holds chunk slot ^ x_swizzle(row).
  const int xrow = wave * 2 * MT + (lane >> 3);
  auto tile_base = [&](int64_t tile, int64_t* r0) {
    const int64_t e = uniform(short_div(tile, tiles_per_part));
    *r0 = (tile - e * tiles_per_part) * kBM;
    return a.X + ((e * a.part_stride + a.part_offset) * a.m + min(*r0, a.m - 1)) * a.d_in;
  };
  // Rows past the partition read its last row, chunks past d_in the row's
  // first chunk: values of that row, which meet zero weights or a zero dZ2.
  auto x_rows = [&](int64_t r0, uint32_t* offset) {
    const int last_row = static_cast<int>(max<int64_t>(min<int64_t>(kBM, a.m - r0), 1)) - 1;
#pragma unroll
    for (int u = 0; u < kXLoads; ++u)
      offset[u] = static_cast<uint32_t>(min(xrow + 8 * u, last_row)) * static_cast<uint32_t>(a.d_in) * 2u;
  };
  auto issue_x = [&](const bf16* Xt, const uint32_t* offset, int step, int stage) {
#pragma unroll
    for (int u = 0; u < kXLoads; ++u) {
      const int kc = step * 8 + ((lane & 7) ^ x_swizzle(xrow + 8 * u));
      if (u * 64 + lane < 16 * MT)
        load_lds16_async(Xt, offset[u] + static_cast<uint32_t>(kc < dchunks ? kc : 0) * 16u,
                         xs_at + static_cast<uint32_t>(stage * kXStage * 2 + (wave * 2 * MT + 8 * u) * 128));
    }
  };
  // Byte offsets into W1F fit 32 bits (hidden * 32 kslices * 2 <= 2^31 + 2^16).
  const uint32_t wlane = static_cast<uint32_t>(wave * NT * 1024 + lane * 16);
  auto issue_w = [&](int s, int buf) {
    uint32_t at = wlane + static_cast<uint32_t>(s) * (kHidden * 64u);
    asm volatile("" : "+v"(at));   // computed here, not kept from tile to tile
    const uint32_t dst = mine_at + static_cast<uint32_t>(buf * kWSlice * 2);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) load_lds16_async(a.W1F, at + nt * 1024u, dst + nt * 1024u);
  };

  if (lane < 16) db2s[wave][lane] = 0.0f;
  int64_t r0;
  const bf16* Xt = tile_base(t, &r0);
  uint32_t xoff[kXLoads];
  x_rows(r0, xoff);
  issue_w(0, 0);
  issue_x(Xt, xoff, 0, 0);
  wait_vmcnt<0>();
  lds_barrier();

  // A tile's sums join those of its run (a block has one or a few) and partition.
  const int32_t runs = a.runs * a.blocks;
  int32_t run = blockIdx.x * a.runs;
  int64_t run_end = a.runs == 1 ? t_end : uniform(linear_block_row(tiles, runs, run + 1));
  bool fresh = true;
  for (; t < t_end; ++t) {
    const int64_t e = uniform(short_div(t, tiles_per_part));

    f32x4 acc[NT][MT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {   // H^T starts from its bias
      f32x4 bias;
#pragma unroll
      for (int i = 0; i < 4; ++i) bias[i] = a.b1[h0 + nt * 16 + 4 * lg + i];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = bias;
    }
    auto compute = [&](int stage, int half, int buf) {
      const bf16* Xs = xs + stage * kXStage + lr * 64 + (((half * 4 + lg) ^ x_swizzle(lr)) << 3);
      const bf16* Ws = mine + buf * kWSlice + lane * 8;
      if constexpr (MT <= NT) {
        bf16x8 xf[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) xf[mt] = load_vec<bf16x8>(Xs + mt * 1024);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const bf16x8 wf = load_vec<bf16x8>(Ws + nt * 512);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = mfma_k32(wf, xf[mt], acc[nt][mt]);
        }
      } else {
        bf16x8 wf[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) wf[nt] = load_vec<bf16x8>(Ws + nt * 512);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const bf16x8 xf = load_vec<bf16x8>(Xs + mt * 1024);
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc[nt][mt] = mfma_k32(wf[nt], xf, acc[nt][mt]);
        }
      }
    };

    // Slice 0 of W1F and the first stage of X are in LDS.
#pragma unroll
    for (int s = 1; s + 1 < WB; ++s)
      if (s < kslices) issue_w(s, s);
    int buf = 0;   // of slice s; the one before it is free
    for (int s = 0; s < kslices; s += 2) {
      const int stage = (s >> 1) & 1;
      // Near the end, where fewer loads were issued, wait for all of them.
      if (s > 0) {
        if (s + max(WB - 2, 1) < kslices) wait_vmcnt<kEvenInFlight>();
        else wait_vmcnt<0>();
        lds_barrier();
      }
      if (s + WB - 1 < kslices) issue_w(s + WB - 1, buf == 0 ? WB - 1 : buf - 1);
      if (s + 2 < kslices) issue_x(Xt, xoff, (s >> 1) + 1, stage ^ 1);
      compute(stage, 0, buf);
      buf = buf + 1 == WB ? 0 : buf + 1;
      if (s + 1 < kslices) {
        if (s + 1 + max(WB - 2, 1) < kslices) wait_vmcnt<kOddInFlight>();
        else wait_vmcnt<0>();
        lds_wait();   // this wave's reads of the slice that is overwritten next
        if (s + WB < kslices) issue_w(s + WB, buf == 0 ? WB - 1 : buf - 1);
        compute(stage, 1, buf);
        buf = buf + 1 == WB ? 0 : buf + 1;
      }
    }

    // Lane indices of what follows, opaque so that no address made from them
    // is kept in registers through the K loop.
    int lr_ = lr, lg_ = lg;
    asm volatile("" : "+v"(lr_), "+v"(lg_));
    // H^T in bf16, and this wave's part of the logits (class 4 lg + i, row lr).
    bf16x4 hb[NT][MT];
    f32x4 z[MT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        bf16x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = static_cast<bf16>(fmaxf(acc[nt][mt][i], 0.0f));
        // Packed at once: two registers follow the four accumulators.
        u32x2 packed = __builtin_bit_cast(u32x2, v);
        asm volatile("" : "+v"(packed));
        hb[nt][mt] = __builtin_bit_cast(bf16x4, packed);
      }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) z[mt] = f32x4{};
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const bf16x4 w2t = load_vec<bf16x4>(a.W2T + lr_ * kHidden + h0 + nt * 16 + 4 * lg_);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) z[mt] = mfma_k16(w2t, hb[nt][mt], z[mt]);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) *reinterpret_cast<f32x4*>(area + mt * 512 + (lg_ * 16 + lr_) * 8) = z[mt];
    lds_barrier();   // the partial logits are there, and every wave is done with the X stages

    const int64_t this_r0 = r0;
    if (t + 1 < t_end) {
      Xt = tile_base(t + 1, &r0);
      x_rows(r0, xoff);
      issue_w(0, 0);
      issue_x(Xt, xoff, 0, 0);
    }

    const int64_t part = e * a.part_stride + a.part_offset;
    if (wave < MT) {   // MT <= 8: one tile per wave
      const int64_t row = this_r0 + wave * 16 + lr_;
      const int label = a.y[part * a.m + min(row, a.m - 1)];
      float b2[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) b2[i] = a.b2[min(4 * lg_ + i, a.classes - 1)];
      f32x4 v = f32x4{};
#pragma unroll
      for (int w = 0; w < kRowsWaves; ++w)
        v += *reinterpret_cast<const f32x4*>(ring + w * (WB * kWSlice) + kWSlice + wave * 512 + (lg_ * 16 + lr_) * 8);
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = 4 * lg_ + i < a.classes ? v[i] + b2[i] : -INFINITY;
        mx = fmaxf(mx, v[i]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      float ex[4], sum = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ex[i] = expf(v[i] - mx);   // 0 past the classes
        sum += ex[i];
      }
      sum += __shfl_xor(sum, 16, 64);
      sum += __shfl_xor(sum, 32, 64);
      bf16x4 dz;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = 4 * lg_ + i;
        const float g =
            (row < a.m && c < a.classes) ? (ex[i] / sum - (c == label ? 1.0f : 0.0f)) * a.inv_m : 0.0f;
        dz[i] = static_cast<bf16>(g);
        dzs[wave][1][c * 16 + lr_] = dz[i];
        const float s = row16_sum(g);
        if (lr_ == 0) db2s[wave][c] += s;
      }
      *reinterpret_cast<bf16x4*>(&dzs[wave][0][lr_ * 16 + 4 * lg_]) = dz;
    }
    wait_vmcnt<0>();   // the next tile's first slices, ahead of this tile's stores
    lds_barrier();

    // The slot's sums so far (dW2^T: class 4 lg + i, unit h0 + 16 nt + lr).
    float* const out = a.partials + (run + e) * a.pstride;
    f32x4* const out_w2 = reinterpret_cast<f32x4*>(out) + wave * NT * 64 + lg_ * 16 + lr_;
    float* const out_b1 = out + kMlpMaxClasses * kHidden + h0 + lr_;
    const bool classes_here = 4 * lg_ < a.classes;
    f32x4 dw2[NT];
    float db1[NT];
    bf16x4 w2p[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      dw2[nt] = f32x4{};
      db1[nt] = 0.0f;
      w2p[nt] = load_vec<bf16x4>(a.W2p + (h0 + nt * 16 + lr_) * kMlpMaxClasses + 4 * lg_);
    }
    if (!fresh) {   // classes past the last group of four: never stored
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) dw2[nt] = out_w2[nt * 64];
    }
    bf16* const dz1 = a.dZ1 + mlp_dz1_index(a.m_pad, kHidden, static_cast<int32_t>(e), this_r0, h0);
    const uint32_t tr = lds_address(area + (4 * lg_ + (lr_ >> 2)) * kTrLd + 4 * (lr_ & 3));
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      if (this_r0 + mt * 16 < a.m_pad) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          *reinterpret_cast<bf16x4*>(area + lr_ * kTrLd + nt * 16 + 4 * lg_) = hb[nt][mt];
        const bf16x4 dz_b = load_vec<bf16x4>(&dzs[mt][0][lr_ * 16 + 4 * lg_]);   // dZ2[lr][4 lg + j]
        const bf16x4 dz_a = load_vec<bf16x4>(&dzs[mt][1][lr_ * 16 + 4 * lg_]);   // dZ2[4 lg + j][lr]
        // H[row 4 lg + j][h0 + 16 nt + lr]: within each 16-lane group, lane i
        // receives element i % 4 of the row pieces addressed by lanes 4 j + i / 4.
        bf16x4v hv[NT];
        read_tr16<NT>(tr, hv);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const bf16x4 hcol = {hv[nt][0], hv[nt][1], hv[nt][2], hv[nt][3]};
          // dH[row 4 lg + i][unit lr]: four consecutive rows of one unit, 8
          // contiguous bytes of dZ1's layout; a wave's store is a 512-byte run.
          const f32x4 dh = mfma_k16(dz_b, w2p[nt], f32x4{});
          bf16x4 g4;
          float gsum = 0.0f;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float g = static_cast<float>(hcol[i]) > 0.0f ? dh[i] : 0.0f;
            gsum += g;
            g4[i] = static_cast<bf16>(g);
          }
          db1[nt] += gsum;
          // dZ1 is streamed: it should not push W1F out of the L2.
          __builtin_nontemporal_store(g4, reinterpret_cast<bf16x4*>(
              dz1 + (static_cast<int64_t>(mt) * kHidden + nt * 16 + lr_) * 16 + 4 * lg_));
          dw2[nt] = mfma_k16(dz_a, hcol, dw2[nt]);
        }
      }
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      if (classes_here) out_w2[nt * 64] = dw2[nt];
      float s = db1[nt];
      s += __shfl_xor(s, 16, 64);
      s += __shfl_xor(s, 32, 64);
      if (lg_ == 0) out_b1[nt * 16] = fresh ? s : out_b1[nt * 16] + s;
    }
    // Every wave has added its tiles' dZ2 (the barrier above): after the last tile of a
    // slot their sum goes to it.
    fresh = t + 1 == run_end || t + 1 == (e + 1) * tiles_per_part;
    if (fresh) {
      if (wave == 0 && lane < 16) {
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < kRowsWaves; ++w) {
          s += db2s[w][lane];
          db2s[w][lane] = 0.0f;
        }
        out[(kMlpMaxClasses + 1) * kHidden + lane] = s;
      }
      if (t + 1 == run_end && t + 1 < t_end) {
        ++run;
        run_end = uniform(linear_block_row(tiles, runs, run + 1));
      }
    }
  }
}

// ---------------------------------------------------------------------------
// wgrad: dW1^T = dZ1^T X per partition (or per split of its rows), block tile 256 hidden x 224 features,
// K = rows in steps of 64.  8 waves: wave (wh, wf) owns hidden rows
// 64 wh .. 64 wh + 63 and features 112 wf .. 112 wf + 111 of the tile (a wave
// whose features all lie past d_in skips its MFMAs).  Both operands travel
// from global memory straight into LDS, one K step ahead, through two buffers
// (every load in the loop is such a load, so they complete in order and the
// per-step waits count them exactly):
//   A (dZ1, 16-row blocked): [4 row blocks][256 hidden][2 halves of 8 rows],
//     half s of hidden h stored at s ^ (((h >> 2) ^ (h >> 3)) & 1); the
//     fragments are plain 16-byte reads.
//   B (X rows): [64 rows][32 chunks of 16 bytes], the tile's 28 feature
//     chunks plus 4 spare, chunk j of row r at slot j ^ g(r) with g(r) even
//     and distinct over rows {0..3, 8..11}, so that the 32-byte row pieces a
//     transposing read gathers spread over the banks.  The fragments (8 rows
//     of one feature per lane) come from two transposing 8-byte reads: within
//     each 16-lane group, lane i receives element i % 4 of the 4-element row
//     pieces addressed by lanes 4 j + i / 4, j = 0..3.
// ---------------------------------------------------------------------------

constexpr int kWgBM = 256, kWgBN = 224, kWgBK = 64, kWgStages = 2;
constexpr int kWgThreads = 512;
constexpr int kWgAChunks = kWgBM * kWgBK / 8;          // 16-byte chunks of an A stage (2048)
constexpr int kWgBRowChunks = kWgBN / 8;               // 28 per X row ...
constexpr int kWgBRowSlots = 32;                       // ... in 32 slots
constexpr int kWgBChunks = kWgBK * kWgBRowSlots;       // 2048
constexpr int kWgStageBytes = (kWgAChunks + kWgBChunks) * 16;
constexpr int kWgALoads = kWgAChunks / kWgThreads, kWgBLoads = kWgBChunks / kWgThreads;
static_assert(kWgALoads * kWgThreads == kWgAChunks && kWgBLoads * kWgThreads == kWgBChunks, "load rounds");
static_assert(kWgStages * kWgStageBytes <= 160 * 1024, "LDS");

__device__ __forceinline__ int wg_half_swizzle(int h) { return ((h >> 2) ^ (h >> 3)) & 1; }
__device__ __forceinline__ int wg_row_swizzle(int r) { return 2 * ((r & 3) | (((r >> 3) & 1) << 2)); }

// The 2 x 7 transposing 8-byte LDS reads of a K half's X fragments: rows OFFSET and OFFSET +
// 2,048 bytes past each address, and the wait for them.  Inline assembly, as for the builtin
// the compiler waits for every outstanding direct-to-LDS load first (it cannot tell the
// buffers apart), which would drain the prefetch; one block, as outside of it the compiler
// takes the results as there from the start and may copy them.  The kernel's own waits and
// barrier order the loads into LDS.
template <int OFFSET>
__device__ __forceinline__ void read_tr16_rows(const uint32_t (&at)[7], bf16x4v (&lo)[7], bf16x4v (&hi)[7]) {
  asm volatile(
      "ds_read_b64_tr_b16 %0, %14 offset:%21\n\tds_read_b64_tr_b16 %7, %14 offset:%22\n\t"
      "ds_read_b64_tr_b16 %1, %15 offset:%21\n\tds_read_b64_tr_b16 %8, %15 offset:%22\n\t"
      "ds_read_b64_tr_b16 %2, %16 offset:%21\n\tds_read_b64_tr_b16 %9, %16 offset:%22\n\t"
      "ds_read_b64_tr_b16 %3, %17 offset:%21\n\tds_read_b64_tr_b16 %10, %17 offset:%22\n\t"
      "ds_read_b64_tr_b16 %4, %18 offset:%21\n\tds_read_b64_tr_b16 %11, %18 offset:%22\n\t"
      "ds_read_b64_tr_b16 %5, %19 offset:%21\n\tds_read_b64_tr_b16 %12, %19 offset:%22\n\t"
      "ds_read_b64_tr_b16 %6, %20 offset:%21\n\tds_read_b64_tr_b16 %13, %20 offset:%22\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(lo[0]), "=&v"(lo[1]), "=&v"(lo[2]), "=&v"(lo[3]), "=&v"(lo[4]), "=&v"(lo[5]), "=&v"(lo[6]),
        "=&v"(hi[0]), "=&v"(hi[1]), "=&v"(hi[2]), "=&v"(hi[3]), "=&v"(hi[4]), "=&v"(hi[5]), "=&v"(hi[6])
      : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[4]), "v"(at[5]), "v"(at[6]), "n"(OFFSET),
        "n"(OFFSET + 2048));
}

// The ring slot that evaluated partition e's gradient goes to.
__device__ __forceinline__ float* ring_slot(const MlpWgradArgs& a, int64_t e) {
  return a.ring + (static_cast<int64_t>(a.plane) * a.n + e * a.part_stride + a.part_offset) * a.ld;
}

__global__ __launch_bounds__(kWgThreads, 1)
void mlp_wgrad_kernel(MlpWgradArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[kWgStages * kWgStageBytes];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int wh = wave & 3, wf = wave >> 2;
  // Work items are the partitions' row splits.  With at least 8 of them, every
  // tile of an item goes to the same XCD (workgroups are dealt to the 8 XCDs
  // round-robin), so its L2 serves the dZ1 rows to all feature tiles and the X
  // rows to all hidden tiles; otherwise the tiles are spread over the chip.
  const int htiles = a.hidden / kWgBM, ftiles = (a.d_in + kWgBN - 1) / kWgBN;
  const int tiles = htiles * ftiles, items = a.n_eval * a.splits;
  const int block = static_cast<int>(blockIdx.x);
  int item, tile;
  if (items >= kXcds) {
    const int local = block / kXcds;
    item = (local / tiles) * kXcds + block % kXcds;
    tile = local % tiles;
    if (item >= items) return;
  } else {
    item = block / tiles;
    tile = block % tiles;
  }
  const int e = item / a.splits, split = item % a.splits;
  const int64_t part = static_cast<int64_t>(e) * a.part_stride + a.part_offset;
  const int hb0 = (tile % htiles) * kWgBM;
  const int i0 = (tile / htiles) * kWgBN;
  const bool active = i0 + wf * (kWgBN / 2) < a.d_in;   // uniform per wave
  const bf16* Xp = a.X + part * a.m * a.d_in;
  const bf16* dz = a.dZ1 + mlp_dz1_index(a.m_pad, a.hidden, e, 0, 0);
  const int64_t steps = a.m_pad / kWgBK;   // at least one per split
  const int k0 = static_cast<int>(split * steps / a.splits);
  const int ksteps = static_cast<int>((split + 1) * steps / a.splits) - k0;

  // A chunk c = u * 512 + tid: row block c / 512, hidden (c % 512) / 2, slot
  // c % 2 holding half (c % 2) ^ swizzle; its source is that half of the row
  // block of dZ1 (a run of 8 KiB per row block in global memory).
  int32_t aoff[kWgALoads];
#pragma unroll
  for (int u = 0; u < kWgALoads; ++u) {
    const int c = u * kWgThreads + tid, rb = c >> 9, h = (c & 511) >> 1;
    aoff[u] = (rb * a.hidden + hb0 + h) * 16 + ((c & 1) ^ wg_half_swizzle(h)) * 8;
  }
  // B chunk c: row c / 32 at slot c % 32, holding feature chunk
  // j = (c % 32) ^ g(row).  Spare chunks (j >= 28) and chunks past d_in read
  // the tile's first chunk of the row; a row past the partition reads its last
  // row: all meet zeros or land in columns that are never used or stored.
  int32_t brow[kWgBLoads], bcol[kWgBLoads];
#pragma unroll
  for (int u = 0; u < kWgBLoads; ++u) {
    const int c = u * kWgThreads + tid, row = c / kWgBRowSlots;
    const int j = (c % kWgBRowSlots) ^ wg_row_swizzle(row);
    const int col = i0 + j * 8;
    brow[u] = row;
    bcol[u] = (j < kWgBRowChunks && col < a.d_in) ? col : i0;
  }
  auto stage_a = [&](int buf) { return reinterpret_cast<bf16*>(smem + buf * kWgStageBytes); };
  auto stage_b = [&](int buf) { return reinterpret_cast<bf16*>(smem + buf * kWgStageBytes + kWgAChunks * 16); };
  auto issue = [&](int ks, int buf) {
    const bf16* dzk = dz + static_cast<int64_t>(k0 + ks) * (kWgBK / 16) * a.hidden * 16;
#pragma unroll
    for (int u = 0; u < kWgALoads; ++u)
      load_lds16(dzk + aoff[u], stage_a(buf) + (u * kWgThreads + wave * 64) * 8);
#pragma unroll
    for (int u = 0; u < kWgBLoads; ++u) {
      const int64_t r = static_cast<int64_t>(k0 + ks) * kWgBK + brow[u];
      load_lds16(Xp + (r < a.m ? r : a.m - 1) * a.d_in + bcol[u], stage_b(buf) + (u * kWgThreads + wave * 64) * 8);
    }
  };

  f32x4 acc[4][7];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int nt = 0; nt < 7; ++nt) acc[mt][nt] = f32x4{};
  // Feature 112 wf + 16 nt + 4 (lr & 3) .. + 3 of the tile sits in chunk 14 wf + 2 nt +
  // ((lr & 3) >> 1), half (lr & 1), of rows 8 lg + (lr >> 2), + 4, + 32 and + 36, whose
  // swizzle is the same.
  const int brow0 = lg * 8 + (lr >> 2);
  uint32_t bat[7];
#pragma unroll
  for (int nt = 0; nt < 7; ++nt)
    bat[nt] = static_cast<uint32_t>(
        (brow0 * kWgBRowSlots + ((14 * wf + 2 * nt + ((lr & 3) >> 1)) ^ wg_row_swizzle(brow0))) * 16 + (lr & 1) * 8);
  auto compute = [&](int buf) {
    const bf16* As = stage_a(buf);
    const uint32_t Bs = lds_address(stage_b(buf));
    uint32_t at[7];
#pragma unroll
    for (int nt = 0; nt < 7; ++nt) at[nt] = Bs + bat[nt];
    auto half = [&](auto kk_) {
      constexpr int kk = decltype(kk_)::value;
      const int rb = kk * 2 + (lg >> 1), half = lg & 1;
      bf16x8 af[4];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const int h = wh * 64 + mt * 16 + lr;
        af[mt] = *reinterpret_cast<const bf16x8*>(&As[((rb * kWgBM + h) * 2 + (half ^ wg_half_swizzle(h))) * 8]);
      }
      bf16x4v lo[7], hi[7];
      read_tr16_rows<kk * 32 * kWgBRowSlots * 16>(at, lo, hi);
#pragma unroll
      for (int nt = 0; nt < 7; ++nt) {
        const bf16x8 bv = {lo[nt][0], lo[nt][1], lo[nt][2], lo[nt][3], hi[nt][0], hi[nt][1], hi[nt][2], hi[nt][3]};
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[mt][nt] = mfma_k32(af[mt], bv, acc[mt][nt]);
      }
    };
    half(std::integral_constant<int, 0>{});
    half(std::integral_constant<int, 1>{});
  };

  issue(0, 0);
  for (int ks = 0; ks < ksteps; ++ks) {
    // This wave's loads of step ks have landed; after the barrier every
    // wave's have, and every wave is done reading the other buffer.
    wait_vmcnt<0>();
    lds_barrier();
    if (ks + 1 < ksteps) issue(ks + 1, (ks + 1) % kWgStages);
    if (active) compute(ks % kWgStages);
  }

  if (!active) return;
  float* slot =
      a.splits == 1 ? ring_slot(a, e) : a.split_sums + static_cast<int64_t>(item) * a.d_in * a.hidden;
#pragma unroll
  for (int nt = 0; nt < 7; ++nt) {
    const int feat = i0 + wf * (kWgBN / 2) + nt * 16 + lr;
    if (feat >= a.d_in) continue;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
      *reinterpret_cast<f32x4*>(slot + static_cast<int64_t>(feat) * a.hidden + hb0 + wh * 64 + mt * 16 + lg * 4) =
          acc[mt][nt];
  }
}

// ---------------------------------------------------------------------------
// reduce: the b1, W2 and b2 parts of the ring slots and, when the weight gradient
// splits its rows, the splits' sums of dW1 (fp64, split order; 16 bytes per thread).
// ---------------------------------------------------------------------------

// Entry j of the rows kernel's sums over partition e (fp64, block order) -> the
// b1, W2 ([hidden][classes] order) and b2 parts of the ring slot.
__device__ __forceinline__ void reduce_small(const MlpSmallParts& r, const MlpWgradArgs& a, int64_t e, int64_t j) {
  if (j >= r.pstride) return;
  const int64_t w1 = static_cast<int64_t>(a.d_in) * a.hidden;
  const int hw = kMlpMaxClasses * a.hidden;
  int64_t at;
  if (j < hw) {   // dW2^T in MFMA order: 16 units x 16 classes, four classes of one unit together
    const int i = static_cast<int>(j);
    const int c = 4 * (i / 64 % 4) + i % 4, h = i / 256 * 16 + i / 4 % 16;
    if (c >= r.classes) return;
    at = w1 + a.hidden + static_cast<int64_t>(h) * r.classes + c;
  } else if (j < hw + a.hidden) {
    at = w1 + (j - hw);
  } else {
    const int c = static_cast<int>(j) - hw - a.hidden;
    if (c >= r.classes) return;
    at = w1 + a.hidden + static_cast<int64_t>(a.hidden) * r.classes + c;
  }
  const int64_t tiles = r.tiles_per_part * a.n_eval;
  const int64_t first = linear_row_block(tiles, r.runs, e * r.tiles_per_part);
  const int64_t last = linear_row_block(tiles, r.runs, (e + 1) * r.tiles_per_part - 1);
  const float* p = r.partials + (first + e) * r.pstride + j;
  const int count = static_cast<int>(last - first) + 1;
  double s = 0.0;
  int b = 0;
  for (; b + 8 <= count; b += 8) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = p[static_cast<int64_t>(b + i) * r.pstride];
#pragma unroll
    for (int i = 0; i < 8; ++i) s += static_cast<double>(v[i]);
  }
  if (b < count) {   // up to 7 more, one latency
    float v[7];
#pragma unroll
    for (int i = 0; i < 7; ++i) v[i] = p[static_cast<int64_t>(min(b + i, count - 1)) * r.pstride];
#pragma unroll
    for (int i = 0; i < 7; ++i)
      if (b + i < count) s += static_cast<double>(v[i]);
  }
  ring_slot(a, e)[at] = static_cast<float>(s);
}

__global__ __launch_bounds__(256)
void mlp_reduce_kernel(MlpWgradArgs a, int fold_blocks) {
  const int64_t e = blockIdx.y;
  if (static_cast<int>(blockIdx.x) >= fold_blocks) {
    reduce_small(a.small, a, e, (blockIdx.x - fold_blocks) * 256 + threadIdx.x);
    return;
  }
  const int64_t q1 = static_cast<int64_t>(a.d_in) * a.hidden;
  const int64_t i = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * 4;
  if (i >= q1) return;
  const float* p = a.split_sums + e * a.splits * q1 + i;
  double sum[4] = {0.0, 0.0, 0.0, 0.0};
  int b = 0;
  for (; b + 4 <= a.splits; b += 4) {
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const f32x4*>(p + (b + u) * q1);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c) sum[c] += static_cast<double>(v[u][c]);
  }
  for (; b < a.splits; ++b) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(p + b * q1);
#pragma unroll
    for (int c = 0; c < 4; ++c) sum[c] += static_cast<double>(v[c]);
  }
  const f32x4 out = {static_cast<float>(sum[0]), static_cast<float>(sum[1]), static_cast<float>(sum[2]),
                     static_cast<float>(sum[3])};
  *reinterpret_cast<f32x4*>(ring_slot(a, e) + i) = out;
}

// Row tiles of the rows kernel by hidden / 256 - 1: MT (16-row groups per tile)
// and the ring's slices, largest tile first.
using RowsKernel = void (*)(MlpRowsArgs);
struct RowsShape { int mt; RowsKernel kernel; };
constexpr int kRowsShapes = 4;
const RowsShape kRows[4][kRowsShapes] = {
    {{6, mlp_rows_kernel<2, 6, 4>}, {4, mlp_rows_kernel<2, 4, 4>}, {2, mlp_rows_kernel<2, 2, 4>},
     {1, mlp_rows_kernel<2, 1, 4>}},
    {{8, mlp_rows_kernel<4, 8, 3>}, {6, mlp_rows_kernel<4, 6, 3>}, {4, mlp_rows_kernel<4, 4, 3>},
     {2, mlp_rows_kernel<4, 2, 3>}},
    {{6, mlp_rows_kernel<6, 6, 2>}, {5, mlp_rows_kernel<6, 5, 2>}, {4, mlp_rows_kernel<6, 4, 2>},
     {2, mlp_rows_kernel<6, 2, 2>}},
    {{6, mlp_rows_kernel<8, 6, 2>}, {5, mlp_rows_kernel<8, 5, 2>}, {4, mlp_rows_kernel<8, 4, 2>},
     {2, mlp_rows_kernel<8, 2, 2>}}};
constexpr int kRowsBlocks = 256;   // one per CU
// Rows whose dW2, db1 and db2 sums share a slot in 32 bits, about.  One slot per block was
// 4,096 rows of a million: error of exact terms 7.3e-8 against 64 bits, 3.3e-8 with five (of
// sums of 1,024 rows 3.9e-8), for 0.2% of the step (more sums to fold).
constexpr int64_t kRowsPerRun = 768;
constexpr int kMaxSplits = 32;

}  // namespace

// The tile that ends first by this estimate of a block's time, in clocks: per K
// slice the MFMAs of its two waves per SIMD or the slice's W1F bytes from L2 at
// 44 bytes per clock, whichever takes longer, then the softmax and dZ1.  It serves
// to compare tiles; with one tile per block, whose slices come from L2 for the first
// time, a kernel takes about twice the estimate.  4 x 5,000 rows at hidden 512: 212
// tiles of 96 rows in 29 us, 160 of 128 in 36.
MlpRowsGrid mlp_rows_grid(int64_t m_pad, int32_t n_eval, int32_t kslices, int32_t hidden) {
  const int nt = hidden / 128;
  MlpRowsGrid best;
  double best_cost = 0.0;
  for (int i = 0; i < kRowsShapes; ++i) {
    const int mt = kRows[hidden / 256 - 1][i].mt;
    MlpRowsGrid g;
    g.shape = i;
    g.tiles_per_part = (m_pad + 16 * mt - 1) / (16 * mt);
    const int64_t tiles = g.tiles_per_part * n_eval;
    g.blocks = static_cast<int32_t>(std::min<int64_t>(kRowsBlocks, tiles));
    const double slice = std::max(32.0 * nt * mt, (nt * 8192.0 + mt * 1024.0) / 44.0) + 200.0;
    const double cost =
        static_cast<double>((tiles + g.blocks - 1) / g.blocks) * (kslices * slice + 270.0 * nt * mt + 6000.0);
    g.runs = static_cast<int32_t>(std::max<int64_t>(1, tiles / g.blocks * 16 * mt / kRowsPerRun));
    if (i == 0 || cost < best_cost) {
      best = g;
      best_cost = cost;
    }
  }
  return best;
}

hipError_t launch_mlp_cast(const MlpCastArgs& a, hipStream_t s) {
  const int64_t items = static_cast<int64_t>(a.kslices) * a.hidden * 4 + static_cast<int64_t>(a.hidden) * kMlpMaxClasses;
  hipLaunchKernelGGL(mlp_cast_kernel, dim3(static_cast<unsigned>((items + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_mlp_rows(const MlpRowsArgs& a, int32_t hidden, int shape, hipStream_t s) {
  if (hidden < 256 || hidden > kMlpMaxHidden || hidden % 256 != 0 || shape < 0 || shape >= kRowsShapes || a.blocks < 1)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(kRows[hidden / 256 - 1][shape].kernel, dim3(a.blocks), dim3(kRowsThreads), 0, s, a);
  return hipGetLastError();
}

// Row splits of the weight gradient.  A partition is hidden / 256 x d_in / 224
// tiles, so few partitions leave most CUs idle: 4 x 5,000 rows at 784 x 512 are 32
// blocks of 79 K steps, 120 us and 5 in the reduce kernel; in the 5 splits that the rule
// picks 34 and 9 us.  Taken is the split that ends first by this estimate, in microseconds:
// rounds of 256 blocks at 1.55 us per K step of 64 rows and 3 us to start and end, then
// the splits' sums written and read at 4 TB/s.  It is not exact: sums that stay in the
// 256 MiB cache cost a quarter of that, a K step of a short run 2.3 us, and 7 splits there
// would take 29 and 10 us.
int mlp_wgrad_splits(int64_t m_pad, int32_t n_eval, int32_t d_in, int32_t hidden) {
  const int64_t steps = m_pad / kWgBK;
  const int64_t tiles = static_cast<int64_t>(hidden / kWgBM) * ((d_in + kWgBN - 1) / kWgBN) * n_eval;
  const double bytes = 8.0 * n_eval * d_in * hidden;
  int best = 1;
  double best_cost = 0.0;
  for (int s = 1; s <= std::min<int64_t>(steps, kMaxSplits); ++s) {
    const double cost = static_cast<double>((tiles * s + 255) / 256) * (static_cast<double>((steps + s - 1) / s) * 1.55 + 3.0) +
                        (s > 1 ? s * bytes / 4e6 + 4.0 : 0.0);
    if (s == 1 || cost < best_cost) {
      best = s;
      best_cost = cost;
    }
  }
  return best;
}

hipError_t launch_mlp_wgrad(const MlpWgradArgs& a, hipStream_t s) {
  const int tiles = (a.hidden / kWgBM) * ((a.d_in + kWgBN - 1) / kWgBN);
  const int items = a.n_eval * a.splits;
  const int parts = items >= kXcds ? (items + kXcds - 1) / kXcds * kXcds : items;
  hipLaunchKernelGGL(mlp_wgrad_kernel, dim3(static_cast<unsigned>(tiles * parts)), dim3(kWgThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_mlp_reduce(const MlpWgradArgs& a, hipStream_t s) {
  const int fold_blocks =
      a.splits > 1 ? static_cast<int>((static_cast<int64_t>(a.d_in) * a.hidden / 4 + 255) / 256) : 0;
  const int small_blocks = static_cast<int>((a.small.pstride + 255) / 256);
  hipLaunchKernelGGL(mlp_reduce_kernel, dim3(fold_blocks + small_blocks, a.n_eval), dim3(256), 0, s, a, fold_blocks);
  return hipGetLastError();
}

}  // namespace pgc
