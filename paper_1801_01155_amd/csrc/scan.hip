// Exclusive prefix sums (reduce-then-scan) and fill kernels for gfx950.
//
// A tile is kThreads x 16 items. Pass 1 reduces each tile to one sum, pass 2
// scans the tile sums in one workgroup, pass 3 rescans each tile with its
// offset. One tile needs pass 3 alone; up to kSumTiles tiles, pass 3 adds up
// the sums before its tile itself (a launch less; launches are what short scans
// cost: 64^3 voxels 3 -> 2, 1000 curves 3 -> 1).
//
// Bound by memory: each wave takes rows of 64 x 16 bytes, loaded and stored as
// they lie, and scans the rows in registers (DPP moves for 32-bit items).
// Against tiles of 4096 staged through LDS: 16.7M items (256^3) 48 -> 32 us,
// 134M (512^3) 450 -> 300 us of kernels (5.3 TB/s).
#include "ls_internal.h"
#include "wave.h"

namespace {

constexpr int kItems = 16;       // per thread
constexpr int kSmallThreads = 256;
constexpr int kLargeThreads = 1024;

template <typename T>
__device__ inline T wave_inclusive_scan(T x) {
  if constexpr (sizeof(T) == 4) {
    return wave_incl_sum(x);
  } else {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      T y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    return x;
  }
}

template <typename T>
__device__ inline T wave_last(T x) {
  return __shfl(x, 63, 64);
}
template <>
__device__ inline uint32_t wave_last(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

template <typename T>
__device__ inline T wave_reduce(T x) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
  return x;
}

// A thread's items: kRows rows of 16 bytes; a wave's row is 64 x 16 bytes in
// memory, its rows follow one another. Zero beyond n.
template <typename T>
struct Rows {
  static constexpr int kPer = 16 / (int)sizeof(T);
  static constexpr int kRows = kItems / kPer;
  T v[kRows][kPer];
};

template <typename T>
__device__ inline int64_t row_index(int64_t base, int r) {
  return base + (int64_t)(threadIdx.x >> 6) * (64 * kItems) +
         (int64_t)(r * 64 + (int)(threadIdx.x & 63)) * Rows<T>::kPer;
}

// whole: all of the tile lies below n and the array is 16-byte aligned.
template <typename T>
__device__ inline void load_rows(const T* in, int64_t base, int64_t n, bool whole, Rows<T>& x) {
  if (whole) {
    uint4 q[Rows<T>::kRows];
#pragma unroll
    for (int r = 0; r < Rows<T>::kRows; ++r)
      q[r] = *reinterpret_cast<const uint4*>(in + row_index<T>(base, r));
#pragma unroll
    for (int r = 0; r < Rows<T>::kRows; ++r) __builtin_memcpy(x.v[r], &q[r], 16);
  } else {
#pragma unroll
    for (int r = 0; r < Rows<T>::kRows; ++r)
#pragma unroll
      for (int j = 0; j < Rows<T>::kPer; ++j) {
        const int64_t i = row_index<T>(base, r) + j;
        x.v[r][j] = i < n ? in[i] : T(0);
      }
  }
}

template <typename T, int kThreads>
__global__ __launch_bounds__(kThreads) void k_tile_reduce(const T* in, int64_t n, bool aligned,
                                                          T* sums) {
  constexpr int kWaves = kThreads / 64;
  __shared__ T wsum[kWaves];
  const int64_t base = (int64_t)blockIdx.x * (kThreads * kItems);
  Rows<T> x;
  load_rows(in, base, n, aligned && base + kThreads * kItems <= n, x);
  T acc = 0;
#pragma unroll
  for (int r = 0; r < Rows<T>::kRows; ++r)
#pragma unroll
    for (int j = 0; j < Rows<T>::kPer; ++j) acc += x.v[r][j];
  acc = wave_reduce(acc);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    T t = 0;
    for (int w = 0; w < kWaves; ++w) t += wsum[w];
    sums[blockIdx.x] = t;
  }
}

// One workgroup of 1024 threads scans `n` tile sums in place (exclusive) and
// writes the grand total to total[0].
template <typename T>
__global__ __launch_bounds__(1024) void k_scan_sums(T* sums, int64_t n, T* total) {
  __shared__ T wsum[16];
  __shared__ T carry_s;
  if (threadIdx.x == 0) carry_s = 0;
  __syncthreads();
  for (int64_t base = 0; base < n; base += 1024) {
    int64_t i = base + threadIdx.x;
    T x = i < n ? sums[i] : T(0);
    T inc = wave_inclusive_scan(x);
    if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = inc;
    __syncthreads();
    T wpre = 0;
    for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) wpre += wsum[w];
    T carry = carry_s;
    if (i < n) sums[i] = carry + wpre + inc - x;
    __syncthreads();
    if (threadIdx.x == 1023) carry_s = carry + wpre + inc;
    __syncthreads();
  }
  if (threadIdx.x == 0) total[0] = carry_s;
}

// kSums: `tiles` holds the tiles' sums (null: a single tile), not their
// exclusive scan; the last tile then also writes the total to out[n].
constexpr int kSumTiles = 1024;

template <typename T, int kThreads, bool kSums>
__global__ __launch_bounds__(kThreads) void k_tile_scan(const T* in, T* out, int64_t n,
                                                        bool aligned, const T* tiles) {
  constexpr int kWaves = kThreads / 64;
  constexpr int kRows = Rows<T>::kRows, kPer = Rows<T>::kPer;
  __shared__ T wsum[kWaves], bsum[kWaves];
  const int wave = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * (kThreads * kItems);
  const bool whole = aligned && base + kThreads * kItems <= n;
  Rows<T> x;
  load_rows(in, base, n, whole, x);
  T before = 0;
  if (kSums && tiles) {
    for (unsigned t = threadIdx.x; t < blockIdx.x; t += kThreads) before += tiles[t];
    before = wave_reduce(before);
  }
  // exclusive scan within the wave, row by row
  T total = 0;
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    T own = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const T v = x.v[r][j];
      x.v[r][j] = own;
      own += v;
    }
    const T inc = wave_inclusive_scan(own);
    const T pre = total + inc - own;
#pragma unroll
    for (int j = 0; j < kPer; ++j) x.v[r][j] += pre;
    total += wave_last(inc);
  }
  if ((threadIdx.x & 63) == 0) {
    wsum[wave] = total;
    bsum[wave] = before;
  }
  __syncthreads();
  T pre = kSums ? T(0) : tiles[blockIdx.x];
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    pre += w < wave ? wsum[w] : T(0);
    if (kSums) pre += bsum[w];
  }
#pragma unroll
  for (int r = 0; r < kRows; ++r)
#pragma unroll
    for (int j = 0; j < kPer; ++j) x.v[r][j] += pre;
  // items beyond n are 0: the last wave's running sum is the total
  if (kSums && blockIdx.x == gridDim.x - 1 && threadIdx.x == kThreads - 1) out[n] = pre + total;
  if (whole) {
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      uint4 q;
      __builtin_memcpy(&q, x.v[r], 16);
      *reinterpret_cast<uint4*>(out + row_index<T>(base, r)) = q;
    }
  } else {
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const int64_t i = row_index<T>(base, r) + j;
        if (i < n) out[i] = x.v[r][j];
      }
  }
}

template <typename T, int kThreads>
int scan_tiles(const T* in, T* out, int64_t n, T* sums, hipStream_t st) {
  const int64_t tiles = (n + kThreads * kItems - 1) / (kThreads * kItems);
  const bool aligned =
      ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
  const dim3 grid((unsigned)tiles), block(kThreads);
  if (tiles == 1) {
    hipLaunchKernelGGL((k_tile_scan<T, kThreads, true>), grid, block, 0, st, in, out, n, aligned,
                       (const T*)nullptr);
    LS_HIP(hipGetLastError());
    return LS_OK;
  }
  hipLaunchKernelGGL((k_tile_reduce<T, kThreads>), grid, block, 0, st, in, n, aligned, sums);
  LS_HIP(hipGetLastError());
  if (tiles <= kSumTiles) {
    hipLaunchKernelGGL((k_tile_scan<T, kThreads, true>), grid, block, 0, st, in, out, n, aligned,
                       (const T*)sums);
    LS_HIP(hipGetLastError());
    return LS_OK;
  }
  hipLaunchKernelGGL((k_scan_sums<T>), dim3(1), dim3(1024), 0, st, sums, tiles, out + n);
  LS_HIP(hipGetLastError());
  hipLaunchKernelGGL((k_tile_scan<T, kThreads, false>), grid, block, 0, st, in, out, n, aligned,
                     (const T*)sums);
  LS_HIP(hipGetLastError());
  return LS_OK;
}

// Large tiles once small ones would be more than kSumTiles: 16.7M items then
// need two launches instead of three and a short sum; below, small tiles fill
// more of the chip.
template <typename T>
int scan_impl(const T* in, T* out, int64_t n, T* sums, hipStream_t st) {
  if (n <= 0) {
    // total of an empty range
    hipLaunchKernelGGL((k_scan_sums<T>), dim3(1), dim3(1024), 0, st, sums, (int64_t)0, out);
    LS_HIP(hipGetLastError());
    return LS_OK;
  }
  if (n <= (int64_t)kSumTiles * kSmallThreads * kItems)
    return scan_tiles<T, kSmallThreads>(in, out, n, sums, st);
  return scan_tiles<T, kLargeThreads>(in, out, n, sums, st);
}

__global__ void k_fill_u32(uint32_t* p, uint32_t v, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

__global__ void k_clear_u32(uint32_t* a, int64_t na, uint32_t* b, int64_t nb, uint32_t* c,
                            int64_t nc) {
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = i0; i < na; i += stride) a[i] = 0u;
  for (int64_t i = i0; i < nb; i += stride) b[i] = 0u;
  for (int64_t i = i0; i < nc; i += stride) c[i] = 0u;
}

__global__ void k_read_words(const uint32_t* src, uint32_t* dst, int n) {
  if ((int)threadIdx.x < n) dst[threadIdx.x] = src[threadIdx.x];
}

}  // namespace

int64_t scan_block_sums_len(int64_t n) {
  return (n + kSmallThreads * kItems - 1) / (kSmallThreads * kItems) + 1;
}

int exclusive_scan_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* sums,
                       hipStream_t st) {
  return scan_impl<uint32_t>(in, out, n, sums, st);
}

int exclusive_scan_u64(const uint64_t* in, uint64_t* out, int64_t n, uint64_t* sums,
                       hipStream_t st) {
  return scan_impl<uint64_t>(in, out, n, sums, st);
}

int fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return LS_OK;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, st, p, v, n);
  LS_HIP(hipGetLastError());
  return LS_OK;
}

int clear_u32(uint32_t* a, int64_t na, uint32_t* b, int64_t nb, uint32_t* c, int64_t nc,
              hipStream_t st) {
  if (!a) na = 0;
  if (!b) nb = 0;
  if (!c) nc = 0;
  const int64_t most = na > nb ? (na > nc ? na : nc) : (nb > nc ? nb : nc);
  if (most <= 0) return LS_OK;
  int64_t blocks = (most + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_clear_u32, dim3((unsigned)blocks), dim3(256), 0, st, a, na, b, nb, c, nc);
  LS_HIP(hipGetLastError());
  return LS_OK;
}

int read_words(const void* dev, void* host, size_t bytes, hipStream_t st) {
  static_assert(kPinnedBytes / 4 <= 64, "one wave copies a slot");
  return read_pinned(host, bytes, st, [&](uint32_t* dst) {
    hipLaunchKernelGGL(k_read_words, dim3(1), dim3(64), 0, st, static_cast<const uint32_t*>(dev),
                       dst, (int)(bytes / 4));
  });
}
