// The row pass over causal logits that the full-span H2O scoring and the entropy profile share.
//
// A workgroup of four waves takes R = 32 NRT query rows of one KV head's group: NRT row tiles of 32, tile T
// being positions i0 + 32 (T % PB) .. of head T / PB, PB = NRT / G.  Each wave holds 64 of them in registers
// (tile32.h) and the head's keys stream through LDS: with eight row tiles the four waves take a quarter of
// the rows each, with four row tiles wave wv takes row half wv % 2 and key half wv / 2 of a tile.  The keys
// are the A operand, so a lane holds one query row and sixteen keys, and its sums are one register each.
// Logits are taken against a fixed per-row reference c = max(logit with the row's own key, logit with
// key 0), both true logits of the row, so x = (z - c) log2(e) / sqrt(d) overflows exp2 only for a key
// more than ~88 natural-log units above it.
//
// Bound: issue of the VALU work on the logits and of the MFMAs, as in the window passes.
#pragma once

#include "tile32.h"

namespace rkv {
namespace {

template <int NRT>
struct CausalRowsLds {
  static constexpr int R = 32 * NRT, RG = NRT / 2, KG = 4 / RG;   // row groups of 64, key groups of a tile
  __attribute__((aligned(16))) uint16_t k[kRing][kTileHalfs];
  float c[R];       // reference logits
  double z[KG][R];   // sum of exp2(x) over the keys of each key group
  double t[KG][R];   // sum of exp2(x) x
};

// Position block (32 queries) and head of a row tile.
template <int NRT, int G>
struct RowTiles {
  static constexpr int PB = NRT / G, kPositions = 32 * PB;
  static_assert(PB >= 1, "a head of the group has at least one row tile");
};

// Sums of the rows of queries i0 .. i0 + 32 PB - 1 (of n_q, at positions L - n_q ..) of the group at qgroup
// ([G][n_q][d]) against the keys of khead up to each row's position, left in sm; rows past n_q get sums
// of no meaning.  kMoment: sm.t too.
template <int NRT, int G, bool kMoment>
__device__ __forceinline__ void causal_rows(const uint16_t* qgroup, int n_q, const uint16_t* khead, int L, int i0, float sl2,
                                            CausalRowsLds<NRT>& sm) {
  constexpr int RG = CausalRowsLds<NRT>::RG, KG = CausalRowsLds<NRT>::KG, PB = RowTiles<NRT, G>::PB;
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), rg = wv % RG, kg = wv / RG;
  bf16x8 q[2][8];
  float ncs[2];
  int last[2];   // the row's position
  double Z[2] = {0.0, 0.0}, T[2] = {0.0, 0.0};
  float Zr[2] = {0.f, 0.f}, Tr[2] = {0.f, 0.f};   // since the ring's last turn
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int rt = 2 * rg + b, i = i0 + 32 * (rt % PB) + l32;
    const uint16_t* row = qgroup + ((size_t)(rt / PB) * n_q + min(i, n_q - 1)) * kHeadDim;
    load_block(i < n_q ? row : nullptr, q[b]);
    last[b] = L - n_q + min(i, n_q - 1);
    const float c = fmaxf(block_dot(q[b], khead + (size_t)last[b] * kHeadDim), block_dot(q[b], khead));
    if (kg == 0 && hf == 0) sm.c[64 * rg + 32 * b + l32] = c;
    ncs[b] = -c * sl2;
  }
  // tiles up to the last position of the workgroup, of this wave; the wave's first position
  const int w0 = i0 + 32 * (2 * rg % PB), w1 = min(n_q, i0 + 32 * ((2 * rg + 1) % PB + 1));
  const int n = (L - n_q + min(n_q, i0 + 32 * PB) - 1) / kTile + 1;
  const int nw = w0 < n_q ? (L - n_q + w1 - 1) / kTile + 1 : 0, first = L - n_q + w0;
  f32x16 accA[2], accB[2];
  hide_all(accB);
  const uint32_t tl = tile_lane();
  // A subtile's sums are taken by themselves first, then those of a turn of the ring, and the turns meet
  // in double precision: a few hundred roundings of small terms added to a large sum would show in
  // the entropies (1.3e-7 against 6e-8 of the subtile sums added up in single precision).
  float zs[2][2], ts[2][2];
  auto exps = [&](const f32x16 (&v)[2], int u) __attribute__((always_inline)) {
    const int b = u >> 4, i = u & 15;
    const float x = fmaf(v[b][i], sl2, ncs[b]);
    const float e = __builtin_amdgcn_exp2f(x);
    if (i < 2) zs[b][i] = e;
    else zs[b][i & 1] += e;
    if constexpr (kMoment) {
      if (i < 2) ts[b][i] = e * x;
      else ts[b][i & 1] = fmaf(e, x, ts[b][i & 1]);
    }
  };
  auto add_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      Zr[b] += zs[b][0] + zs[b][1];
      if constexpr (kMoment) Tr[b] += ts[b][0] + ts[b][1];
    }
  };
  auto turn = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      Z[b] += (double)Zr[b];
      Zr[b] = 0.f;
      if constexpr (kMoment) {
        T[b] += (double)Tr[b];
        Tr[b] = 0.f;
      }
    }
  };
  // a subtile of keys k0 .. k0 + 31, with the exponentials of the one before it
  auto step = [&](const uint16_t* tile, int sub, int k0, f32x16 (&cur)[2], const f32x16 (&prev)[2]) __attribute__((always_inline)) {
    tile_step<true>(tile, tl, sub, q, cur, [&](int u) __attribute__((always_inline)) { exps(prev, u); });
    add_sums();
    keep_here(Zr);
    if constexpr (kMoment) keep_here(Tr);
    if (k0 + 31 > first) {   // keys past a row's position take no part
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (k0 + acc_row(i) + 4 * hf > last[b]) cur[b][i] = kHidden;
    }
  };
  const uint32_t lds0 = lds_addr(&sm.k[0][0]);
  stream_tiles<kTileDma>(n, [&](int t, int buf) __attribute__((always_inline)) {
    issue_tile(khead, t * kTile, L, lds0 + buf * (kTileHalfs * 2), wv);
  }, [&](auto buf, int t) __attribute__((always_inline)) {
    constexpr int b = decltype(buf)::value;
    if (PB > 1 && t >= nw) return;   // past the wave's rows, not yet past the workgroup's
    const int k0 = t * kTile;
    if constexpr (KG == 1) {
      step(sm.k[b], 0, k0, accA, accB);
      step(sm.k[b], 1, k0 + 32, accB, accA);
    } else if constexpr ((b & 1) == 0) {
      step(sm.k[b], kg, k0 + 32 * kg, accA, accB);
    } else {
      step(sm.k[b], kg, k0 + 32 * kg, accB, accA);
    }
    if constexpr (b == kRing - 1) turn();
  });
  if (KG == 1 || (nw & 1) == 0) {
#pragma unroll
    for (int u = 0; u < 32; ++u) exps(accB, u);
  } else {
#pragma unroll
    for (int u = 0; u < 32; ++u) exps(accA, u);
  }
  add_sums();
  turn();
  sm.z[kg][64 * rg + lane] = halves_sum(Z);
  if constexpr (kMoment) sm.t[kg][64 * rg + lane] = halves_sum(T);
  tile_barrier();
}

// Launch shape of the row pass over `rows` query rows of each of n_jobs KV heads.  Four row tiles a
// workgroup below 1024 workgroups of eight, which leave the 512 resident ones unevenly filled (16 jobs of
// 1030 rows and 9001 keys: 371 us against 395; 8 jobs of 8000 rows: 31 against 39; 48 of 3100: 192 against 201),
// eight from there on, whose key fragments serve twice the rows (64 jobs of 4400 rows: 208 against 212; 256
// jobs of 16384: 2300 against 2490).
inline bool causal_rows_small(int n_jobs, int64_t rows) { return (rows + 255) / 256 * n_jobs < 1024; }
// Its order: the longest items first where the lengths differ and the launch is short (48 jobs of 3100
// queries: 180 us against 200; 64 of 1100: 200 against 208), job by job elsewhere (256 jobs of 4096
// queries: 2300 against 2360; the last 515 of 9001: 371 against 391).
inline bool causal_rows_by_job(int64_t items, int n_q, int L) { return items >= 4096 || 2 * (int64_t)n_q <= L; }

}  // namespace
}  // namespace rkv
