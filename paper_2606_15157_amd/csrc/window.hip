// Window scoring on gfx950 where the pipelined kernel does not apply (more than 64 slices of 128 keys per
// job, eight row tiles: G * ceil(w / 32) > 4, inputs that are not 16-byte aligned) or is the slower one (many
// jobs of padded rows or of few slices; window_faster has the rule).  Per (sequence, layer, KV head)
// job the scores are those of the pipelined kernel (Section 2.1's SnapKV and H2O rules):
//   A[g][j] = sum_i softmax_j(Q[g,i] . K[j] / sqrt(d)), S = mean_g maxpool(A[g]) or mean_g A[g],
// computed in two passes over the keys instead of one pass with a cross-workgroup exchange.
//
// Both passes (four waves; tile32.h) hold 64 of the job's R = 32 NRT window rows (the rows of every
// head of the group, padded) per wave in registers and stream the keys through LDS in 64-key tiles:
// with eight row tiles the four waves take a quarter of the rows each, with four row tiles wave wv
// takes row half wv % 2 and key half wv / 2 of a tile.  The MFMAs of a 32-key subtile run beside the
// exponentials of the one before, across tiles too; tiles with masked pairs only overwrite the
// masked logits in between.
//
// window_rows_kernel<NRT>: one workgroup per job (per part of its keys when there are few jobs:
//   the columns kernel then adds the parts' row sums).  The keys are the A operand, so a lane holds
//   one window row of each block and some keys, and the row's sum and reference are one register each: e =
//   exp2((z - c_r) log2(e) / sqrt(d)) against a fixed per-row reference c_r = max(logit with the
//   row's own key, logit with key 0).  c_r and the row sum go to the workspace.
// window_cols_kernel<NRT>: one workgroup per (job, range of 128-key slices).  The window rows are
//   the A operand, so a lane holds one key and some rows of each block, with two numbers of each row in
//   registers; its probabilities are summed over a block's rows in registers and
//   the per-head column sums give the slice's pooled and unpooled scores and slice-edge sums in
//   the layout of the pipelined kernel, so the same selection (with its slice-border pool repair)
//   follows.  Jobs, ranges and tiles run in the reverse of the rows kernel's order, so that the keys it
//   read last are still in the 256 MB last-level cache.
// Sums run in a fixed order (the only atomic sets a status bit): results are reproducible.
//
// Either kernel takes its logits from 32x32x16 MFMA or, for the prompts that the pipelined kernel could take,
// from 16x16x32 (fewer roundings).
//
// Bound: issue of the exponentials and MFMAs (per 64 logits 16 cycles of multiply-add, exponential
// and addition, beside 16 of the matrix pipe, half of which hold back the VALU too), at the clock the
// power limit leaves (1.6 GHz).  With eight row tiles the rows pass has the VALU busy 0.84 and the matrix pipe 0.74
// of the time, the columns pass 0.62 and 0.49, its waves waiting (barriers, stores) for 0.29.  At 960 jobs of
// 256 rows and 32768 keys the rows pass takes 1.93 ms (2.38 with 16x16x32 MFMA and 32 rows per wave, 1.09
// PFLOP/s now) and the columns pass 2.39 ms (3.04).  Four row tiles are bound by the second reading of the keys: 128 jobs of 20011 keys, 656 MB
// a pass, 140 and 128 us (150 and 216).
#include <hip/hip_runtime.h>

#include <math.h>

#include "tile32.h"

namespace rkv {
namespace {

// Window row r of a job: query head g = r / tpr and window index ii = r % tpr (tpr = rows per
// head in the padded layout); valid when g < G and ii < w.
struct WinRow {
  int g, ii;
  bool valid;
};
__device__ __forceinline__ WinRow win_row(int r, int tpr, int G, int w) {
  WinRow x;
  x.g = r / tpr;
  x.ii = r - x.g * tpr;
  x.valid = x.g < G && x.ii < w;
  return x;
}

// The key tiles kt0 + kDir t, t = 0 .. n - 1, of a key head through the ring.
template <int kDir, typename Body>
__device__ __forceinline__ void stream_keys(const uint16_t* khead, int L, int kt0, int n, uint16_t (*sK)[kTileHalfs],
                                            int wv, Body&& body) {
  const uint32_t lds0 = lds_addr(&sK[0][0]);
  stream_tiles<kTileDma>(n, [&](int t, int buf) __attribute__((always_inline)) {
    issue_tile(khead, (kt0 + kDir * t) * kTile, L, lds0 + buf * (kTileHalfs * 2), wv);
  }, body);
}

// How the rows kernel takes a wave's 64 window rows: the keys are the A operand, so a lane holds one row of each
// block (kBlocks blocks of kRows rows) and some keys, and the row's reference and sums are one register each.
// Sums: a subtile's exponentials by themselves first, then those of a turn of the ring, and the turns in
// double precision, so the rounding of many small terms added to a large one stays out of them.
//
// WideSums, 32x32x16 MFMA: e = exp2(x), x = z log2(e)/sqrt(d) - c log2(e)/sqrt(d).
struct WideSums {
  static constexpr int kBlocks = 2, kRows = 32;
  f32x16 acc[2][2];   // two subtiles in flight
  bf16x8 q[2][8];
  int last[2];        // last visible key
  float nc[2], zs[2][4], Zr[2], sl2;
  double Z[2];
  __device__ __forceinline__ void load(int b, const uint16_t* row) { load_block(row, q[b]); }
  __device__ __forceinline__ float dot(int b, const uint16_t* key) const { return block_dot(q[b], key); }
  __device__ __forceinline__ void reference(int b, float c) { nc[b] = -c * sl2; }
  template <int X>
  __device__ __forceinline__ void hide() { hide_all(acc[X]); }
  template <int X>
  __device__ __forceinline__ void exps(int u) {
    const int b = u >> 4, i = u & 15;
    const float e = __builtin_amdgcn_exp2f(fmaf(acc[X][b][i], sl2, nc[b]));
    if (i < 4) zs[b][i] = e;
    else zs[b][i & 3] += e;
  }
  template <int X>   // a subtile into acc[X], beside the exponentials of acc[1 - X]
  __device__ __forceinline__ void step(const uint16_t* tile, int sub) {
    tile_step<true>(tile, tile_lane(), sub, q, acc[X], [&](int u) __attribute__((always_inline)) { exps<1 - X>(u); });
  }
  template <int X>   // hides the keys of a subtile at k0 past a row's position (or the prompt)
  __device__ __forceinline__ void mask(int k0) {
    const int hf = (threadIdx.x >> 5) & 1;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (k0 + acc_row(i) + 4 * hf > last[b]) acc[X][b][i] = kHidden;
  }
  __device__ __forceinline__ void keep() { keep_here(Zr); }
  // the wave's row sums, over the lanes of a row, to out[0 .. 63]
  __device__ __forceinline__ void put(double* out) const { out[threadIdx.x & 63] = halves_sum(Z); }
};
// FineSums, 16x16x32 MFMA: half as many roundings of z, and accumulators that start from -c (see FineRows).
struct FineSums {
  static constexpr int kBlocks = 4, kRows = 16;
  f32x4 acc[2][2][4];
  bf16x8 q[4][4];
  int last[4];
  f32x4 nc[4];        // -c in every element
  float zs[4][4], Zr[4], sl2;
  double Z[4];
  __device__ __forceinline__ void load(int b, const uint16_t* row) { load_block16(row, q[b]); }
  __device__ __forceinline__ float dot(int b, const uint16_t* key) const { return block_dot16(q[b], key); }
  __device__ __forceinline__ void reference(int b, float c) { nc[b] = {-c, -c, -c, -c}; }
  template <int X>
  __device__ __forceinline__ void hide() {
#pragma unroll
    for (int u = 0; u < 32; ++u) acc[X][u >> 4][(u >> 2) & 3][u & 3] = kHidden;
  }
  template <int X>
  __device__ __forceinline__ void exps(int u) {
    const int kh = u >> 4, b = (u >> 2) & 3, i = u & 3;
    const float e = __builtin_amdgcn_exp2f(acc[X][kh][b][i] * sl2);
    if (kh == 0) zs[b][i] = e;
    else zs[b][i] += e;
  }
  template <int X>
  __device__ __forceinline__ void step(const uint16_t* tile, int sub) {
    tile_step16<true>(tile, tile_lane16(), sub, q, nc, acc[X], [&](int u) __attribute__((always_inline)) { exps<1 - X>(u); });
  }
  template <int X>
  __device__ __forceinline__ void mask(int k0) {
    const int lg = (threadIdx.x >> 4) & 3;
#pragma unroll
    for (int u = 0; u < 32; ++u) {
      const int kh = u >> 4, b = (u >> 2) & 3, i = u & 3;
      if (k0 + 16 * kh + 4 * lg + i > last[b]) acc[X][kh][b][i] = kHidden;
    }
  }
  __device__ __forceinline__ void keep() { asm volatile("" : "+v"(Zr[0]), "+v"(Zr[1]), "+v"(Zr[2]), "+v"(Zr[3])); }
  __device__ __forceinline__ void put(double* out) const {   // lane group lg ends with block lg
    const int lane = threadIdx.x & 63;
    double s = 0.0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      double z = Z[b] + __shfl_xor(Z[b], 16);
      z += __shfl_xor(z, 32);
      if (lane >> 4 == b) s = z;
    }
    out[lane] = s;
  }
};

template <int NRT, typename Rows>
__global__ __launch_bounds__(256, 2) void window_rows_kernel(const PrefillLaunch P) {
  constexpr int R = NRT * 32, RG = NRT / 2, KG = 4 / RG;   // row groups of 64, key groups of a tile
  __shared__ __attribute__((aligned(16))) uint16_t sK[kRing][kTileHalfs];
  __shared__ double sZ[KG][R];
  __shared__ float sC[R];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), rg = wv % RG, kg = wv / RG;
  const int L = P.seq_len, w = P.window, G = P.group, Hq = P.n_q_heads, Hkv = P.n_kv_heads, B = P.batch;
  const int tpr = P.row_tiles_per_group * 32;
  const int parts = P.window_parts, job = blockIdx.x / parts, part = blockIdx.x - job * parts;
  const int h = job % Hkv, s = (job / Hkv) % B, slot = job / (Hkv * B);
  const PrefillLayer& ly = P.layer[slot];
  const uint16_t* khead = ly.k + (size_t)(s * Hkv + h) * L * kHeadDim;
  const uint16_t* qjob = ly.q + (size_t)(s * Hq + h * G) * w * kHeadDim;   // [G][w][d]
  // this workgroup's key tiles [t0, t0 + n) (part `part` of the job's tiles)
  const int n_tiles = (L + kTile - 1) / kTile, per_part = (n_tiles + parts - 1) / parts;
  const int t0 = min(n_tiles, part * per_part), n = min(n_tiles, t0 + per_part) - t0;

  // the wave's rows 64 rg .., their references and last visible keys
  Rows rows;
  rows.sl2 = P.scale_log2;
#pragma unroll
  for (int b = 0; b < Rows::kBlocks; ++b) {
    const int r = 64 * rg + Rows::kRows * b + lane % Rows::kRows;
    const WinRow x = win_row(r, tpr, G, w);
    rows.load(b, x.valid ? qjob + (size_t)(x.g * w + x.ii) * kHeadDim : nullptr);
    rows.last[b] = x.valid ? L - w + x.ii : L - 1;
    const float c = fmaxf(rows.dot(b, khead + (size_t)rows.last[b] * kHeadDim), rows.dot(b, khead));
    if (kg == 0 && lane < Rows::kRows) sC[r] = c;
    rows.reference(b, c);
    rows.Z[b] = 0.0;
    rows.Zr[b] = 0.f;
  }
  rows.template hide<1>();
  auto add_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < Rows::kBlocks; ++b) rows.Zr[b] += (rows.zs[b][0] + rows.zs[b][1]) + (rows.zs[b][2] + rows.zs[b][3]);
  };
  auto turn = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < Rows::kBlocks; ++b) {
      rows.Z[b] += (double)rows.Zr[b];
      rows.Zr[b] = 0.f;
    }
  };
  // a subtile of keys k0 .. k0 + 31 into accumulators X, with the exponentials of the one before it
  auto step = [&](auto X, const uint16_t* tile, int sub, int k0) __attribute__((always_inline)) {
    constexpr int x = decltype(X)::value;
    rows.template step<x>(tile, sub);
    add_sums();
    rows.keep();
    if (k0 + 31 > L - w) rows.template mask<x>(k0);
  };
  const std::integral_constant<int, 0> kA{};
  const std::integral_constant<int, 1> kB{};
  stream_keys<1>(khead, L, t0, n, sK, wv, [&](auto buf, int t) __attribute__((always_inline)) {
    constexpr int b = decltype(buf)::value;
    const int k0 = (t0 + t) * kTile;
    if constexpr (KG == 1) {
      step(kA, sK[b], 0, k0);
      step(kB, sK[b], 1, k0 + 32);
    } else if constexpr ((b & 1) == 0) {
      step(kA, sK[b], kg, k0 + 32 * kg);
    } else {
      step(kB, sK[b], kg, k0 + 32 * kg);
    }
    if constexpr (b == kRing - 1) turn();
  });
  if (KG == 1 || (n & 1) == 0) {
#pragma unroll
    for (int u = 0; u < 32; ++u) rows.template exps<1>(u);
  } else {
#pragma unroll
    for (int u = 0; u < 32; ++u) rows.template exps<0>(u);
  }
  // sums over the lane halves and the key groups; the row's log2 normaliser (one part), or the part's
  // row sum and, from part 0, the reference (several parts: the columns kernel adds them)
  add_sums();
  turn();
  rows.put(&sZ[kg][64 * rg]);
  tile_barrier();
  if (tid < R) {
    double zd = sZ[0][tid];
#pragma unroll
    for (int k = 1; k < KG; ++k) zd += sZ[k][tid];
    const float z = (float)zd;
    if (part == 0) P.ncl[(size_t)job * R + tid] = win_row(tid, tpr, G, w).valid ? sC[tid] : __builtin_inff();
    if (parts == 1) P.lam[(size_t)job * R + tid] = z;
    else P.stats[((size_t)job * parts + part) * R + tid] = z;
  }
  if (blockIdx.x == 0 && tid == 0 && P.first_group) P.counters[0] = 0u;   // the call's status word
}

// How the columns kernel takes a wave's 64 window rows: they are the A operand, so a lane holds one key and some
// rows of each block, and two numbers of every row, made of its reference logit c and its row sum z.
//
// WideRows, 32x32x16 MFMA: p = exp2(x), x = z_rj log2(e)/sqrt(d) - Lambda_r, the row's log2 normaliser.
struct WideRows {
  f32x16 acc[2][2];   // two subtiles in flight
  bf16x8 q[2][8];
  f32x4 nl[2][4];     // -Lambda
  float cs[2][4];     // column sums of a block
  float sl2;
  static __device__ __forceinline__ float2 numbers(float c, float z, float sl2) { return {-add_log2(c * sl2, z), 0.f}; }
  template <typename Row>   // row(r): the wave's row r (0 .. 63) in memory, or null
  __device__ __forceinline__ void load(Row&& row) {
#pragma unroll
    for (int b = 0; b < 2; ++b) load_block(row(32 * b + (int)(threadIdx.x & 31)), q[b]);
  }
  __device__ __forceinline__ void stats(const float* a, const float*) {
    const int hf = (threadIdx.x >> 5) & 1;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int u = 0; u < 4; ++u) nl[b][u] = *reinterpret_cast<const f32x4*>(a + 32 * b + 8 * u + 4 * hf);
  }
  template <int X>
  __device__ __forceinline__ void hide() { hide_all(acc[X]); }
  template <int X>
  __device__ __forceinline__ void exps(int u) {
    const int b = u >> 4, i = u & 15;
    const float e = __builtin_amdgcn_exp2f(fmaf(acc[X][b][i], sl2, nl[b][i >> 2][i & 3]));
    if (i < 4) cs[b][i] = e;
    else cs[b][i & 3] += e;
  }
  template <int X>   // a subtile into acc[X], beside the exponentials of acc[1 - X]
  __device__ __forceinline__ void step(const uint16_t* tile, int sub) {
    tile_step<false>(tile, tile_lane(), sub, q, acc[X], [&](int u) __attribute__((always_inline)) { exps<1 - X>(u); });
  }
  template <int X, typename Seen>   // seen(key of the subtile, row): hides the others
  __device__ __forceinline__ void mask(Seen&& seen) {
    const int l32 = threadIdx.x & 31, hf = (threadIdx.x >> 5) & 1;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (!seen(l32, b, acc_row(i) + 4 * hf)) acc[X][b][i] = kHidden;
  }
  // column sums of the subtile to sum0 (the wave's first row tile) and sum1, of both to sum0 if `pair`
  __device__ __forceinline__ void put(float* sum0, float* sum1, bool pair) const {
    const int l32 = threadIdx.x & 31, hf = (threadIdx.x >> 5) & 1;
    const float c0 = (cs[0][0] + cs[0][1]) + (cs[0][2] + cs[0][3]), c1 = (cs[1][0] + cs[1][1]) + (cs[1][2] + cs[1][3]);
    if (pair) {
      const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(c0 + c1), __float_as_uint(c0 + c1), false, false);
      if (hf == 0) sum0[l32] = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    } else {
      const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(c0), __float_as_uint(c1), false, false);
      (hf ? sum1 : sum0)[l32] = __uint_as_float(p[0]) + __uint_as_float(p[1]);   // lane half hf: block hf
    }
  }
};
// FineRows, 16x16x32 MFMA: p = exp2(x) w_r, x = (z_rj - c_r) log2(e)/sqrt(d) from accumulators that start from
// -c_r, with the weight w_r = 1 / z_r.  That is the pipelined kernel's arithmetic: no number of the size of
// Lambda is rounded, a logit is rounded half as often, and near the reference, where the large probabilities
// are, against a small number.  Its error is the pipelined kernel's: 1.00 of it over 22 padded and short layouts
// of 16 prompts each (0.97 to 1.03 a layout; batch 3, L = 3331, w = 27, two heads a group: 1.20e-7 and 1.21e-7).
// Accumulators from 0 left 1.04 to 1.15 of it, and WideRows 1.54e-7 there for 4 % less time.
struct FineRows {
  f32x4 acc[2][2][4];
  bf16x8 q[4][4];
  f32x4 nc[4], wt[4];   // -c, w
  float cs[2][2];       // column sums of a key half and row tile
  float sl2;
  static __device__ __forceinline__ float2 numbers(float c, float z, float) {
    return {-c, c < __builtin_inff() ? 1.f / z : 0.f};
  }
  template <typename Row>
  __device__ __forceinline__ void load(Row&& row) {
#pragma unroll
    for (int b = 0; b < 4; ++b) load_block16(row(16 * b + (int)(threadIdx.x & 15)), q[b]);
  }
  __device__ __forceinline__ void stats(const float* a, const float* w) {
    const int lg = (threadIdx.x >> 4) & 3;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      nc[b] = *reinterpret_cast<const f32x4*>(a + 16 * b + 4 * lg);
      wt[b] = *reinterpret_cast<const f32x4*>(w + 16 * b + 4 * lg);
    }
  }
  template <int X>
  __device__ __forceinline__ void hide() {
    mask<X>([](int, int, int) { return false; });
  }
  template <int X>
  __device__ __forceinline__ void exps(int u) {
    const int kh = u >> 4, b = (u >> 2) & 3, i = u & 3;
    const float e = __builtin_amdgcn_exp2f(acc[X][kh][b][i] * sl2);
    if ((u & 7) == 0) cs[kh][b >> 1] = e * wt[b][i];
    else cs[kh][b >> 1] = fmaf(e, wt[b][i], cs[kh][b >> 1]);
  }
  template <int X>
  __device__ __forceinline__ void step(const uint16_t* tile, int sub) {
    tile_step16<false>(tile, tile_lane16(), sub, q, nc, acc[X], [&](int u) __attribute__((always_inline)) { exps<1 - X>(u); });
  }
  template <int X, typename Seen>
  __device__ __forceinline__ void mask(Seen&& seen) {
    const int l16 = threadIdx.x & 15, lg = (threadIdx.x >> 4) & 3;
#pragma unroll
    for (int u = 0; u < 32; ++u) {
      const int kh = u >> 4, b = (u >> 2) & 3, i = u & 3;
      if (!seen(16 * kh + l16, b >> 1, 16 * (b & 1) + 4 * lg + i)) acc[X][kh][b][i] = kHidden;
    }
  }
  __device__ __forceinline__ void put(float* sum0, float* sum1, bool pair) const {
    // over the four lane groups of a key: lane group lg then has key half lg / 2 and row tile lg % 2
    auto half = [&](float a, float b) __attribute__((always_inline)) {
      const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
      return __uint_as_float(p[0]) + __uint_as_float(p[1]);
    };
    const int l16 = threadIdx.x & 15, lg = (threadIdx.x >> 4) & 3, k = 16 * (lg >> 1) + l16;
    if (pair) {
      const float c = half(cs[0][0] + cs[0][1], cs[1][0] + cs[1][1]);
      const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(c), __float_as_uint(c), false, false);
      if ((lg & 1) == 0) sum0[k] = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    } else {
      const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(half(cs[0][0], cs[1][0])),
                                                      __float_as_uint(half(cs[0][1], cs[1][1])), false, false);
      ((lg & 1) ? sum1 : sum0)[k] = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    }
  }
};

template <int NRT, typename Rows>
__global__ __launch_bounds__(256, 2) void window_cols_kernel(const PrefillLaunch P) {
  constexpr int R = NRT * 32, NT = 256, RG = NRT / 2, KG = 4 / RG;
  __shared__ __attribute__((aligned(16))) uint16_t sK[kRing][kTileHalfs];
  // column sums of a slice's keys, per 32-row block (an odd number of row tiles per head) or per
  // 64-row pair of blocks (an even number: both belong to one head); two slices in flight
  constexpr int kPad = 4, kColRow = kSlice + 2 * kPad;   // rows with a zero margin at both ends
  __shared__ float sCol[2][NRT][kColRow];
  __shared__ __attribute__((aligned(16))) float sA[R], sB[R];   // the rows' numbers
  const int tid = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), rg = wv % RG, kg = wv / RG;
  const int L = P.seq_len, w = P.window, G = P.group, Hq = P.n_q_heads, Hkv = P.n_kv_heads, B = P.batch;
  const int nsl = P.n_slices, NTH = P.row_tiles_per_group, tpr = NTH * 32;
  const bool pair = NTH % 2 == 0;
  const int per_head = pair ? NTH / 2 : NTH;   // sCol rows of a head
  const int ranges = P.window_ranges, per_range = (nsl + ranges - 1) / ranges;
  const int block = gridDim.x - 1 - blockIdx.x;   // what the rows kernel read last comes first
  const int job = block / ranges, range = block - job * ranges;
  const int b0 = min(nsl, range * per_range), b1 = min(nsl, b0 + per_range), n = 2 * (b1 - b0);
  const int h = job % Hkv, s = (job / Hkv) % B, slot = job / (Hkv * B);
  const PrefillLayer& ly = P.layer[slot];
  const bool snap = ly.rule == RKV_SNAPKV;
  const uint16_t* khead = ly.k + (size_t)(s * Hkv + h) * L * kHeadDim;
  const uint16_t* qjob = ly.q + (size_t)(s * Hq + h * G) * w * kHeadDim;
  const float sl2 = P.scale_log2, inv_g = 1.f / (float)G;
  const int npre = L - w, ph = P.pool_half;
  if (n <= 0) return;

  if (tid < 2 * NRT * 2 * kPad) {
    const int o = tid % (2 * kPad);
    (&sCol[0][0][0])[tid / (2 * kPad) * kColRow + (o < kPad ? o : kSlice + o)] = 0.f;
  }
  Rows rows;
  rows.sl2 = sl2;
  bool over = false;
  if (tid < R) {
    float z;   // the row's sum (several parts: theirs added in part order, rounded once)
    if (P.window_parts == 1) {
      z = P.lam[(size_t)job * R + tid];
    } else {
      double zd = 0.0;
      for (int p = 0; p < P.window_parts; ++p) zd += (double)P.stats[((size_t)job * P.window_parts + p) * R + tid];
      z = (float)zd;
    }
    // padding and overflowing rows: reference +inf, every probability 0
    float c = P.ncl[(size_t)job * R + tid];
    if (!(z < __builtin_inff())) {
      over = win_row(tid, tpr, G, w).valid;
      z = 1.f;
      c = __builtin_inff();
    }
    const float2 n = Rows::numbers(c, z, sl2);
    sA[tid] = n.x;
    sB[tid] = n.y;
  }
  if (range == 0) {
    // A row whose sum overflows, in one part or over all of them: the job is rescored exactly before selection.
    const int any = __syncthreads_or(over);
    if (tid == 0) {
      P.counters[(size_t)kCounterStride * (1 + job) + 1] = any ? 1u : 0u;
      if (any) atomicOr(P.counters, RKV_STATUS_REPAIRED);
    }
  }
  rows.load([&](int r) __attribute__((always_inline)) {
    const WinRow x = win_row(64 * rg + r, tpr, G, w);
    return x.valid ? qjob + (size_t)(x.g * w + x.ii) * kHeadDim : nullptr;
  });
  tile_barrier();
  rows.stats(sA + 64 * rg, sB + 64 * rg);
  // Scores of slice b from the column sums in buffer sb.  The common forms (one sCol row per head, no
  // mask border in the slice, a 7-wide pool where pooled) take one wave pair for the keys, every head
  // of a key in one thread, and the other pair for the slice-edge sums.  Their pool windows are cut by
  // the zero margins of sCol instead of clamped indices: the sums are non-negative, so a margin never
  // is the maximum, and the maximum of the bit patterns is the maximum of the values.
  auto store = [&](int b, int sb) __attribute__((always_inline)) {
    int tid = threadIdx.x;   // opaque: no per-thread address is kept across the loop
    asm volatile("" : "+v"(tid));
    const float(*col)[kColRow] = sCol[sb];
    const int cbase = b * kSlice;
    float* Srow = P.S + (size_t)job * L + cbase;
    if (per_head == 1 && cbase + kSlice <= npre && (!snap || ph == 3)) {
      const int t2 = tid ^ (sb << 7);   // the wave pairs take turns
      if (t2 < kSlice) {
        // head pairs: two roundings of a mean of four, where one head after another takes three
        const float* c = &col[0][kPad + t2];
        auto pool = [](const float* x) __attribute__((always_inline)) {
          const uint32_t* u = reinterpret_cast<const uint32_t*>(x);
          return __uint_as_float(max(max(max(u[-3], u[-2]), max(u[-1], u[0])), max(max(u[1], u[2]), u[3])));
        };
        float su = 0.f, sc = 0.f;
        if (snap) {
#pragma unroll 2
          for (int g = 0; g + 1 < G; g += 2, c += 2 * kColRow) {
            su += c[0] + c[kColRow];
            sc += pool(c) + pool(c + kColRow);
          }
          if (G & 1) {
            su += c[0];
            sc += pool(c);
          }
          Srow[t2] = sc * inv_g;
          if (P.want_unpooled) P.Su[(size_t)job * L + cbase + t2] = su * inv_g;
        } else {
#pragma unroll 2
          for (int g = 0; g + 1 < G; g += 2, c += 2 * kColRow) su += c[0] + c[kColRow];
          if (G & 1) su += c[0];
          Srow[t2] = su * inv_g;
        }
      } else if (snap && t2 - kSlice < 12 * G) {   // offsets 0 .. 5 and 122 .. 127 of every head
        const int e = t2 - kSlice, g = e / 12, o = e - 12 * g;
        P.edge[((size_t)job * nsl + b) * G * 12 + e] = col[g][kPad + (o < 6 ? o : kSlice - 12 + o)];
      }
      return;
    }
    auto head = [&](int g, int kl) {
      float v = col[g * per_head][kPad + kl];
      for (int u = 1; u < per_head; ++u) v += col[g * per_head + u][kPad + kl];
      return v;
    };
    // thread = (key, query-head half)
    const int kl = tid >> 1, kk = cbase + kl;
    const int g0 = (tid & 1) * ((G + 1) >> 1), g1 = min(G, g0 + ((G + 1) >> 1));
    float su = 0.f, sc = 0.f;
    if (kk < L) {
      // max-pool window [lo, hi] inside the slice and the prefix [0, L - w); clamping a
      // neighbour into it repeats a member (for window keys the pooled value is not used)
      const int lo = max(kk - ph, cbase) - cbase;
      const int hi = max(min(min(kk + ph, cbase + kSlice - 1), npre - 1) - cbase, lo);
      for (int g = g0; g < g1; ++g) {
        su += head(g, kl);
        if (snap) {
          float m = 0.f;
          for (int u = 0; u <= 2 * ph; ++u) m = fmaxf(m, head(g, min(max(kl - ph + u, lo), hi)));
          sc += m;
        }
      }
    }
    su += dpp_pair(su);   // the other head half's sum (lane ^ 1)
    sc += dpp_pair(sc);
    if ((tid & 1) == 0 && kk < L) {
      su *= inv_g;
      Srow[kl] = snap && kk < npre ? sc * inv_g : su;
      if (snap && P.want_unpooled) P.Su[(size_t)job * L + kk] = su;
    }
    if (snap && ph > 0) {   // slice-edge column sums per head: offsets [0, 2 ph) and [128 - 2 ph, 128)
      const int E = 4 * ph, twoP = 2 * ph;
      float* ed = P.edge + ((size_t)job * nsl + b) * G * E;
      for (int e2 = tid; e2 < G * E; e2 += NT) {
        const int g = e2 / E, o = e2 - g * E;
        const int kl2 = o < twoP ? o : kSlice - twoP + (o - twoP);
        ed[e2] = (cbase + kl2 < L) ? head(g, kl2) : 0.f;
      }
    }
  };
  // the column sums of a subtile: key offset kb of the slice in buffer sb (both constants)
  auto put = [&](int sb, int kb) __attribute__((always_inline)) {
    if (pair) rows.put(&sCol[sb][rg][kPad + kb], nullptr, true);
    else rows.put(&sCol[sb][2 * rg][kPad + kb], &sCol[sb][2 * rg + 1][kPad + kb], false);
  };
  rows.template hide<1>();
  // the subtile at key ka into accumulators X, beside the exponentials of the one before it, whose sums then
  // go to (sb, kb)
  auto step = [&](auto X, const uint16_t* tile, int sub, int ka, int sb, int kb) __attribute__((always_inline)) {
    constexpr int x = decltype(X)::value;
    rows.template step<x>(tile, sub);
    put(sb, kb);
    if (ka + 31 > L - w)   // keys past a row's position (or the prompt) take no part
      rows.template mask<x>([&](int key, int rt, int r) __attribute__((always_inline)) {
        return ka + key <= L - w + 32 * ((2 * rg + rt) % NTH) + r;   // window index of the row tile's first row, plus r
      });
  };
  const std::integral_constant<int, 0> kA{};
  const std::integral_constant<int, 1> kB{};
  // Tiles and slices run downwards.  The slice of tile t is in column buffer (t / 2) % 2.  Its last sums are written during the next
  // slice's first tile, so its scores are stored in that slice's second tile, after the barrier; the
  // buffer is written again from the first tile of the slice after that.  (The first step of all puts
  // zeros where the second slice comes.)
  stream_keys<-1>(khead, L, 2 * b1 - 1, n, sK, wv, [&](auto buf, int t) __attribute__((always_inline)) {
    constexpr int b = decltype(buf)::value, pb = (b + kRing - 1) % kRing;   // this tile's buffer, the one before
    const int ka = (2 * b1 - 1 - t) * kTile;
    if constexpr (KG == 1) {
      step(kA, sK[b], 0, ka, pb / 2, b % 2 * kTile + 32);
      step(kB, sK[b], 1, ka + 32, b / 2, pb % 2 * kTile);
    } else if constexpr (b % 2 == 0) {
      step(kA, sK[b], kg, ka + 32 * kg, pb / 2, b % 2 * kTile + 32 * kg);
    } else {
      step(kB, sK[b], kg, ka + 32 * kg, pb / 2, b % 2 * kTile + 32 * kg);
    }
    if (b % 2 == 1 && t >= 3) store(b1 - t / 2, 1 - b / 2);
  });
#pragma unroll
  for (int u = 0; u < 32; ++u) rows.template exps<1>(u);   // n is even: the last subtile's
  const int sb = (b1 - 1 - b0) & 1;
  put(sb, KG == 1 ? 32 : 32 * kg);
  tile_barrier();
  store(b0, sb);
}

template <int NRT>
int launch_window_nrt(const PrefillLaunch& P, int n_jobs, hipStream_t st) {
  const unsigned rows = (unsigned)(n_jobs * P.window_parts), cols = (unsigned)((int64_t)n_jobs * P.window_ranges);
  if constexpr (NRT == 4) {
    if (P.n_slices <= kPipeMaxSlices) {   // prompts the pipelined kernel could take: FineRows has why
      window_rows_kernel<NRT, FineSums><<<rows, 256, 0, st>>>(P);
      window_cols_kernel<NRT, FineRows><<<cols, 256, 0, st>>>(P);
      return (int)hipGetLastError();
    }
  }
  window_rows_kernel<NRT, WideSums><<<rows, 256, 0, st>>>(P);
  window_cols_kernel<NRT, WideRows><<<cols, 256, 0, st>>>(P);
  return (int)hipGetLastError();
}

}  // namespace

int launch_window(const PrefillLaunch& P, int row_tiles, void* stream) {
  const int n_jobs = P.batch * P.n_window * P.n_kv_heads;
  if (n_jobs <= 0) return 0;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  return row_tiles <= 4 ? launch_window_nrt<4>(P, n_jobs, st) : launch_window_nrt<8>(P, n_jobs, st);
}

}  // namespace rkv
