// Logit tiles on 32x32x16 bf16 MFMA for the kernels that stream rows (keys, or queries) through
// LDS past a 64-row block each wave holds in registers (window, full-span and entropy scoring).
//
// A streamed tile is 64 rows of 128 bf16 (16 KiB), brought in by LDS DMA into a ring of four
// buffers, three tiles ahead, shared by the four waves of a workgroup: one barrier per tile.
// Every fragment a wave reads from LDS (32 rows x 16 columns, one ds_read_b128 per lane) feeds the
// two MFMAs of its two 32-row blocks, 64 matrix-pipe cycles: at two waves per SIMD the CU's LDS is
// then read about half of the time.  (With 16x16x32 MFMA and 32 rows per wave every read fed 32
// cycles, which saturated the LDS.)
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

#include <type_traits>

#include "lds_dma.h"
#include "rkv_internal.h"

namespace rkv {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kTile = 64;                            // streamed rows per tile
constexpr int kTileHalfs = kTile * kHeadDim;         // 16-bit values of a tile
constexpr int kRing = 4;                             // tile buffers of a workgroup
constexpr int kTileDma = 4;                          // DMA instructions per wave and tile
constexpr float kHidden = -3.402823466e38f;          // logit of a hidden pair (finite: 0 times it is 0): its exponential is 0

// Workgroup barrier for data handed over through LDS only: this wave's LDS operations retire, then
// s_barrier; vector memory operations stay in flight.
__device__ __forceinline__ void tile_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt 0
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Rows [row0, row0 + 64) of `rows` ([n][128] bf16) into the tile buffer at LDS address lds; rows
// from n on repeat row n - 1.  Wave wv of four moves instructions I = wv + 4 u (rows 4 I .. 4 I + 3,
// 1 KiB each): lane l fills row 4 I + l / 16, chunk position l % 16, with source chunk
// (l % 16) ^ (row % 16) (row % 16 = 4 wv + l / 16 for every u), the swizzle tile_frag reads.  Rows
// that are not 16-byte aligned (a view into a larger buffer) go through registers: the buffer is
// then complete at this wave's next tile_barrier, as is every DMA the wave issued earlier, whatever
// wait_tile counts.
__device__ __forceinline__ void issue_tile(const uint16_t* rows, int row0, int n, uint32_t lds, int wv) {
  const int lane = threadIdx.x & 63, r4 = 4 * wv + (lane >> 4);
  const uint32_t chunk = (uint32_t)((lane & 15) ^ r4) * 16u;
  const bool aligned = ((uintptr_t)rows & 15) == 0;
  if (aligned && row0 + kTile <= n) {
    const char* base = reinterpret_cast<const char*>(rows + (size_t)row0 * kHeadDim) + 1024 * wv;
    const uint32_t off = (uint32_t)(lane >> 4) * 256u + chunk;
    dma16s_pair(base, off, lds + 1024u * wv);
    dma16s_pair(base + 8192, off, lds + 1024u * wv + 8192u);
  } else if (!aligned) {
    u32x4 v[kTileDma];
#pragma unroll
    for (int u = 0; u < kTileDma; ++u) {
      const int row = min(row0 + 16 * u + r4, n - 1);
      __builtin_memcpy(&v[u], reinterpret_cast<const char*>(rows + (size_t)row * kHeadDim) + chunk, 16);
    }
#pragma unroll
    for (int u = 0; u < kTileDma; ++u)
      *(__attribute__((address_space(3))) u32x4*)(uintptr_t)(lds + 1024u * (wv + 4 * u) + 16u * lane) = v[u];
    wait_vmcnt<0>();
  } else {
#pragma unroll
    for (int u = 0; u < kTileDma; ++u) {
      const int row = min(row0 + 16 * u + r4, n - 1);
      dma16(reinterpret_cast<const char*>(rows + (size_t)row * kHeadDim) + chunk, lds + 1024u * (wv + 4 * u));
    }
  }
}

// Waits until a tile's own DMA (kDma instructions a tile) is in, with `later` tiles (0, 1 or at least
// 2) issued after it.
template <int kDma>
__device__ __forceinline__ void wait_tile(int later) {
  if (later >= 2) wait_vmcnt<2 * kDma>();
  else if (later == 1) wait_vmcnt<kDma>();
  else wait_vmcnt<0>();
}

// Runs `body(buffer, t)` for the streamed tiles t = 0 .. n - 1, each in buffer t % kRing (a compile-time
// constant) after `issue(t, buffer)` requested it with kDma DMA instructions a wave.  Tile t + 3 is
// requested once every wave is past tile t - 1, whose buffer it takes.
template <int kDma, typename Issue, typename Body>
__device__ __forceinline__ void stream_tiles(int n, Issue&& issue, Body&& body) {
#pragma unroll
  for (int t = 0; t < kRing - 1; ++t)
    if (t < n) issue(t, t);
  auto one = [&](auto buf, int t) __attribute__((always_inline)) {
    constexpr int b = decltype(buf)::value;
    wait_tile<kDma>(n - 1 - t);
    tile_barrier();
    if (t + kRing - 1 < n) issue(t + kRing - 1, (b + kRing - 1) % kRing);
    body(buf, t);
  };
#pragma unroll 1
  for (int t = 0; t < n; t += kRing) {
    one(std::integral_constant<int, 0>{}, t);
    if (t + 1 < n) one(std::integral_constant<int, 1>{}, t + 1);
    if (t + 2 < n) one(std::integral_constant<int, 2>{}, t + 2);
    if (t + 3 < n) one(std::integral_constant<int, 3>{}, t + 3);
  }
}

// The same with the tiles two at a time, 2 p and 2 p + 1 in buffers 2 (p % 2) and 2 (p % 2) + 1, and
// `body(p % 2, p)`: one barrier for both, so that waves which take a tile of the pair each work side by side.
// A last tile without a partner is requested twice.
template <int kDma, typename Issue, typename Body>
__device__ __forceinline__ void stream_pairs(int n, Issue&& issue, Body&& body) {
  const int np = (n + 1) / 2;
  auto request = [&](int p, int at) __attribute__((always_inline)) {
    issue(2 * p, 2 * at);
    issue(min(2 * p + 1, n - 1), 2 * at + 1);
  };
  request(0, 0);
  auto one = [&](auto at, int p) __attribute__((always_inline)) {
    constexpr int b = decltype(at)::value;
    wait_tile<kDma>(0);
    tile_barrier();
    if (p + 1 < np) request(p + 1, 1 - b);   // every wave is past pair p - 1
    body(at, p);
  };
#pragma unroll 1
  for (int p = 0; p < np; p += 2) {
    one(std::integral_constant<int, 0>{}, p);
    if (p + 1 < np) one(std::integral_constant<int, 1>{}, p + 1);
  }
}

// Byte offset inside a tile of this lane's fragment of k-step st (rows sub * 32 + lane % 32, 16-byte
// chunk 2 st + lane / 32): tile_lane() ^ (32 st), plus 8192 sub.
__device__ __forceinline__ uint32_t tile_lane() {
  const uint32_t r = threadIdx.x & 31, hf = (threadIdx.x >> 5) & 1;
  return r * 256u + ((r & 15) ^ hf) * 16u;
}
__device__ __forceinline__ bf16x8 tile_frag(const uint16_t* tile, uint32_t tl, int sub, int st) {
  return *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(tile) + (tl ^ (32u * st)) + 8192u * sub);
}

// Registers of a wave's own rows: row lane % 32 of a 32-row block, chunk 2 st + lane / 32 (the A and
// the B operand have the same form).  A null row reads as zeros.
__device__ __forceinline__ void load_block(const uint16_t* row, bf16x8 (&f)[8]) {
  const int hf = (threadIdx.x >> 5) & 1;
#pragma unroll
  for (int st = 0; st < 8; ++st) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (row) v = *reinterpret_cast<const u32x4*>(row + 8 * (2 * st + hf));
    f[st] = __builtin_bit_cast(bf16x8, v);
  }
}
// The two bf16 in a dword, which is taken by value: __builtin_bit_cast of a vector's element reads element 0
// whatever the index (seen with the compiler of ROCm 7.2).
__device__ __forceinline__ bf16x2 bf16_pair(uint32_t v) { return __builtin_bit_cast(bf16x2, v); }
// Dot product of this lane's row (in f) with another row in memory, both halves of the row summed.
__device__ __forceinline__ float block_dot(const bf16x8 (&f)[8], const uint16_t* row) {
  const int hf = (threadIdx.x >> 5) & 1;
  float a = 0.f;
#pragma unroll
  for (int st = 0; st < 8; ++st) {
    const u32x4 x = *reinterpret_cast<const u32x4*>(row + 8 * (2 * st + hf));
    const u32x4 y = __builtin_bit_cast(u32x4, f[st]);
#pragma unroll
    for (int u = 0; u < 4; ++u) a = __builtin_amdgcn_fdot2_f32_bf16(bf16_pair(x[u]), bf16_pair(y[u]), a, false);
  }
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(a), false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

// Register i of an accumulator is row acc_row(i) + 4 (lane / 32) of its 32 x 32 tile (its column is
// lane % 32).
__device__ __forceinline__ constexpr int acc_row(int i) { return 8 * (i >> 2) + (i & 3); }

// One 32-row subtile of the streamed tile against the wave's two blocks, software-pipelined with the
// VALU work on the previous subtile's logits: step j reads fragment j + 2, runs fragment j's two
// MFMAs and 4 of the 32 values `value(u)` (u = block * 16 + register) of the previous subtile; a
// scheduling barrier closes the step.  The first four values cover the first reads' latency.
// kStreamA: the streamed rows are the A operand (accumulator rows), else the B operand.
template <bool kStreamA, typename Value>
__device__ __forceinline__ void tile_step(const uint16_t* tile, uint32_t tl, int sub, const bf16x8 (&own)[2][8],
                                          f32x16 (&acc)[2], Value&& value) {
  bf16x8 f[3];
  f[0] = tile_frag(tile, tl, sub, 0);
  f[1] = tile_frag(tile, tl, sub, 1);
#pragma unroll
  for (int u = 0; u < 4; ++u) value(u);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (j + 2 < 8) f[(j + 2) % 3] = tile_frag(tile, tl, sub, j + 2);
    const f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < 2; ++b)
      acc[b] = kStreamA ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[j % 3], own[b][j], j == 0 ? z : acc[b], 0, 0, 0)
                        : __builtin_amdgcn_mfma_f32_32x32x16_bf16(own[b][j], f[j % 3], j == 0 ? z : acc[b], 0, 0, 0);
    if (j < 7) {
#pragma unroll
      for (int u = 4 * j + 4; u < 4 * j + 8; ++u) value(u);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The same with 16x16x32 MFMA: the wave's rows are four blocks of 16 (own[b][st]: row lane % 16, chunk 4 st +
// lane / 16), the streamed subtile two of 16.  Register i of acc[kh][b] is row 4 (lane / 16) + i of the A
// operand (block b, or part kh of the subtile with kStreamA), its column row lane % 16 of the other.  Half as
// many roundings of a logit as with 32x32x16, for twice the MFMA issue.  Values are numbered
// u = 16 kh + 4 b + i.
__device__ __forceinline__ uint32_t tile_lane16() {
  const uint32_t r = threadIdx.x & 15, lg = (threadIdx.x >> 4) & 3;
  return r * 256u + (r ^ lg) * 16u;
}
__device__ __forceinline__ void load_block16(const uint16_t* row, bf16x8 (&f)[4]) {
  const int lg = (threadIdx.x >> 4) & 3;
#pragma unroll
  for (int st = 0; st < 4; ++st) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (row) v = *reinterpret_cast<const u32x4*>(row + 8 * (4 * st + lg));
    f[st] = __builtin_bit_cast(bf16x8, v);
  }
}
// Dot product of this lane's row with another row in memory, over the row's four lane groups.
__device__ __forceinline__ float block_dot16(const bf16x8 (&f)[4], const uint16_t* row) {
  const int lg = (threadIdx.x >> 4) & 3;
  float a = 0.f;
#pragma unroll
  for (int st = 0; st < 4; ++st) {
    const u32x4 x = *reinterpret_cast<const u32x4*>(row + 8 * (4 * st + lg));
    const u32x4 y = __builtin_bit_cast(u32x4, f[st]);
#pragma unroll
    for (int u = 0; u < 4; ++u) a = __builtin_amdgcn_fdot2_f32_bf16(bf16_pair(x[u]), bf16_pair(y[u]), a, false);
  }
  a += __shfl_xor(a, 16);
  return a + __shfl_xor(a, 32);
}
// Accumulators of block b start as start[b].
template <bool kStreamA, typename Value>
__device__ __forceinline__ void tile_step16(const uint16_t* tile, uint32_t tl, int sub, const bf16x8 (&own)[4][4],
                                            const f32x4 (&start)[4], f32x4 (&acc)[2][4], Value&& value) {
  auto frag = [&](int j) __attribute__((always_inline)) {   // (kh, st) = (j / 4, j % 4)
    return *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(tile) + (tl ^ (64u * (j & 3))) + 4096u * (j >> 2) + 8192u * sub);
  };
  bf16x8 f[3];
  f[0] = frag(0);
  f[1] = frag(1);
#pragma unroll
  for (int u = 0; u < 4; ++u) value(u);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (j + 2 < 8) f[(j + 2) % 3] = frag(j + 2);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const f32x4 c = (j & 3) == 0 ? start[b] : acc[j >> 2][b];
      acc[j >> 2][b] = kStreamA ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[j % 3], own[b][j & 3], c, 0, 0, 0)
                                : __builtin_amdgcn_mfma_f32_16x16x32_bf16(own[b][j & 3], f[j % 3], c, 0, 0, 0);
    }
    if (j < 7) {
#pragma unroll
      for (int u = 4 * j + 4; u < 4 * j + 8; ++u) value(u);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Sums that only a later iteration reads: without this the compiler sinks the additions, and the
// exponentials that feed them, out of the MFMA steps they are interleaved with.
__device__ __forceinline__ void keep_here(float (&z)[2]) { asm volatile("" : "+v"(z[0]), "+v"(z[1])); }
// x plus the value of another lane of its 16-lane row.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false));
}
// The value of lane ^ 1.
__device__ __forceinline__ float dpp_pair(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xf, 0xf, false));
}

// The sums of a wave's 64 rows over the two lane halves: lane half hf returns block hf's.
__device__ __forceinline__ double halves_sum(const double (&a)[2]) {
  const int hf = (threadIdx.x >> 5) & 1;
  const double other = __shfl_xor(hf ? a[0] : a[1], 32);
  return (hf ? a[1] : a[0]) + other;
}

// c + log2(z) for z >= 1, rounded once.  The logarithm is taken of the mantissa: of z itself (a row sum
// in the thousands) its last bit is 1e-6, an error that all rows of like sums share.
__device__ __forceinline__ float add_log2(float c, float z) {
  return (float)((double)c + (double)__builtin_amdgcn_frexp_expf(z) + (double)__builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(z)));
}

__device__ __forceinline__ void hide_all(f32x16 (&a)[2]) {
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) a[b][i] = kHidden;
}

// Work item of a grid with `per_job` workgroups for each of n_jobs jobs whose workgroups stream the same
// rows; item 0 of every job is its longest.  by_job: eight jobs at a time, one per XCD (workgroups go round
// the eight XCDs), so that a job's rows are fetched into one L2 cache; otherwise the longest items of all
// jobs come first, which ends the launch evenly.
struct JobItem {
  int job, item;
};
__device__ __forceinline__ JobItem job_item(int block, int n_jobs, int per_job, bool by_job) {
  if (!by_job) return {block % n_jobs, block / n_jobs};
  const int first = block / (8 * per_job) * 8, r = block - first * per_job, n = min(8, n_jobs - first);
  return {first + r % n, r / n};
}

}  // namespace
}  // namespace rkv
