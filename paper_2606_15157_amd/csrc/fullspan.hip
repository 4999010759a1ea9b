// H2O prefill with full-span accumulation on gfx950: the score of key j is the group mean of the
// attention it receives from every prompt query t >= j (H2O's accumulated attention, Section 2.1),
//   S[h, j] = (1/G) sum_g sum_{t >= j} softmax_j(q[hG+g, t] . k[h, .] / sqrt(d)) over keys <= t.
// Two passes over the causal logits, no atomics, fixed summation order:
//
// fullspan_rows_kernel: one workgroup per (job, block of query positions), the row pass of
//   causal_rows.h over 128 or 256 query rows of the group.  The row's log2 normaliser Lambda_t =
//   c_t log2(e)/sqrt(d) + log2(sum_j exp2(x_tj)) goes to the workspace.  A non-finite normaliser (a key
//   beyond ~88 natural-log units above the reference c_t) sets status bit 1.
// fullspan_cols_kernel: one workgroup per (job, key block), each wave with 64 keys in registers (tile32.h).
//   The group's query rows at or after the block stream through LDS in tiles of 64 positions of one
//   head, with their normalisers, from the last position down (the workgroups of a job start together on
//   the same rows, which stay in their XCD's L2 cache).  The keys are the A operand, so a lane holds one
//   query row, with its normaliser in one register, and sixteen keys of each block: it sums
//   p = exp2(x - Lambda_t) per key in 32 registers, and the 32 lanes of a key meet once at the end.
// Bound: issue of the exponentials and MFMAs, each logit twice.  32 jobs of 8192 queries and four heads: rows
// 1.04 ms (1.56 with 16x16x32 MFMA, 32 rows a wave and 128-key tiles through registers), columns 0.95 (2.05),
// 1.1 TFLOP of causal logits each; the error of the scores against 64 bits 1.7e-7 (8e-6, in columns summed
// over thousands of terms a lane).
// Jobs here are the full-span ones: job = (slot * B + b) * Hkv + h with slot >= n_window.
#include <hip/hip_runtime.h>

#include <math.h>

#include "causal_rows.h"

namespace rkv {
namespace {

template <int NRT, int G>
__global__ __launch_bounds__(256, 2) void fullspan_rows_kernel(const PrefillLaunch P, int by_job) {
  constexpr int R = 32 * NRT, PB = RowTiles<NRT, G>::PB, kPos = RowTiles<NRT, G>::kPositions;
  __shared__ CausalRowsLds<NRT> sm;
  const int tid = threadIdx.x;
  const int L = P.seq_len, Hq = P.n_q_heads, Hkv = P.n_kv_heads, B = P.batch;
  const int nqb = (L + kPos - 1) / kPos;
  const JobItem it = job_item(blockIdx.x, B * Hkv * P.n_full, nqb, by_job != 0);
  const int t0 = (nqb - 1 - it.item) * kPos;   // the longest rows first
  const int job = B * Hkv * P.n_window + it.job;
  const int h = job % Hkv, s = (job / Hkv) % B, slot = job / (Hkv * B);
  const PrefillLayer& ly = P.layer[slot];
  causal_rows<NRT, G, false>(ly.q + (size_t)(s * Hq + h * G) * L * kHeadDim, L, ly.k + (size_t)(s * Hkv + h) * L * kHeadDim, L,
                             t0, P.scale_log2, sm);
  if (tid < R) {
    double zd = 0.0;
#pragma unroll
    for (int k = 0; k < CausalRowsLds<NRT>::KG; ++k) zd += sm.z[k][tid];
    const float z = (float)zd;
    const int rt = tid >> 5, t = t0 + 32 * (rt % PB) + (tid & 31);
    if (t < L) {
      if (!(z < __builtin_inff())) atomicOr(P.counters, 2u);
      P.lamf[((size_t)it.job * G + rt / PB) * L + t] = add_log2(sm.c[tid] * P.scale_log2, z);
    }
  }
}

// KG waves share the query rows of a key group of 64: one takes every row (256 keys a workgroup), two a subtile
// of each tile, four a subtile of each pair of tiles.
template <int G, int KG>
__global__ __launch_bounds__(256, 2) void fullspan_cols_kernel(const PrefillLaunch P) {
  constexpr int RG = 4 / KG, kKeys = 64 * RG, kDma = kTileDma + 1;
  __shared__ __attribute__((aligned(16))) uint16_t sQ[kRing][kTileHalfs];
  __shared__ __attribute__((aligned(16))) float sLam[kRing][4][kTile];   // every wave brings in its own copy
  __shared__ float sCol[KG][kKeys];
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), rg = wv % RG, kg = wv / RG;
  const int L = P.seq_len, Hq = P.n_q_heads, Hkv = P.n_kv_heads, B = P.batch;
  const int nkb = (L + kKeys - 1) / kKeys;
  const JobItem it = job_item(blockIdx.x, B * Hkv * P.n_full, nkb, false);
  const int job = B * Hkv * P.n_window + it.job;
  const int h = job % Hkv, s = (job / Hkv) % B, slot = job / (Hkv * B);
  const PrefillLayer& ly = P.layer[slot];
  const int j0 = it.item * kKeys, jw = j0 + 64 * rg;   // the workgroup's, the wave's first key
  const uint16_t* khead = ly.k + (size_t)(s * Hkv + h) * L * kHeadDim;
  const uint16_t* qbase = ly.q + (size_t)(s * Hq + h * G) * L * kHeadDim;   // the group's first head
  const float* lamj = P.lamf + (size_t)it.job * G * L;

  bf16x8 key[2][8];
#pragma unroll
  for (int b = 0; b < 2; ++b)   // keys past the prompt are unused
    load_block(khead + (size_t)min(jw + 32 * b + l32, L - 1) * kHeadDim, key[b]);
  // tile t: positions 64 (p_last - t / G) .. of head t % G, down to the position tile of the workgroup's
  // (of the wave's) first key
  const int p_last = (L - 1) / kTile;
  const int n = (p_last - j0 / kTile + 1) * G, nw = max(0, p_last - jw / kTile + 1) * G;
  const float sl2 = P.scale_log2;
  f32x16 accA[2], accB[2], col[2];
  hide_all(accB);
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) col[b][i] = 0.f;
  float nA = 0.f, nB = 0.f;   // minus the normaliser of this lane's row in accA, accB
  auto exps = [&](const f32x16 (&v)[2], float nl, int u) __attribute__((always_inline)) {
    const int b = u >> 4, i = u & 15;
    col[b][i] += __builtin_amdgcn_exp2f(fmaf(v[b][i], sl2, nl));
  };
  const uint32_t tl = tile_lane();
  // the subtile of rows at positions t0 .. t0 + 31, beside the exponentials of the one before it
  auto step = [&](const uint16_t* tile, const float* lam, int sub, int t0, f32x16 (&cur)[2], float& ncur,
                  const f32x16 (&prev)[2], float nprev) __attribute__((always_inline)) {
    ncur = -lam[32 * sub + l32];
    tile_step<false>(tile, tl, sub, key, cur, [&](int u) __attribute__((always_inline)) { exps(prev, nprev, u); });
    asm volatile("" : "+v"(col[0]), "+v"(col[1]));   // as keep_here
    if (t0 < jw + 63 || t0 + 31 >= L) {
      // near the diagonal or past the prompt: hidden pairs add nothing, whatever the row's normaliser.  Such
      // a subtile is summed at once and leaves hidden logits behind.
      const int t = t0 + l32;
#pragma unroll
      for (int u = 0; u < 32; ++u) {
        const int b = u >> 4, i = u & 15;
        const float e = __builtin_amdgcn_exp2f(fmaf(cur[b][i], sl2, ncur));
        col[b][i] += t >= L || jw + 32 * b + acc_row(i) + 4 * hf > t ? 0.f : e;
      }
      hide_all(cur);
      ncur = 0.f;
    }
  };
  const uint32_t lds0 = lds_addr(&sQ[0][0]), lam0 = lds_addr(&sLam[0][wv][0]);
  auto issue = [&](int t, int buf) __attribute__((always_inline)) {
    const int g = t % G, t0 = (p_last - t / G) * kTile;
    issue_tile(qbase + (size_t)g * L * kHeadDim, t0, L, lds0 + buf * (kTileHalfs * 2), wv);
    dma4(lamj + (size_t)g * L + min(t0 + lane, L - 1), lam0 + buf * (4 * kTile * 4));
  };
  if constexpr (KG == 4) {
    stream_pairs<kDma>(n, issue, [&](auto at, int p) __attribute__((always_inline)) {
      const int sub = kg & 1, t = 2 * p + (kg >> 1), buf = 2 * decltype(at)::value + (kg >> 1);
      if (t >= nw) return;   // before the wave's keys, or a last tile without a partner
      const int t0 = (p_last - t / G) * kTile + 32 * sub;
      if constexpr (decltype(at)::value == 0) step(sQ[buf], &sLam[buf][wv][0], sub, t0, accA, nA, accB, nB);
      else step(sQ[buf], &sLam[buf][wv][0], sub, t0, accB, nB, accA, nA);
    });
  } else {
    stream_tiles<kDma>(n, issue, [&](auto buf, int t) __attribute__((always_inline)) {
      constexpr int b = decltype(buf)::value;
      if (t >= nw) return;   // before the wave's keys, not yet before the workgroup's
      const int t0 = (p_last - t / G) * kTile, sub = kg;
      const float* lam = &sLam[b][wv][0];
      if constexpr (KG == 1) {
        step(sQ[b], lam, 0, t0, accA, nA, accB, nB);
        step(sQ[b], lam, 1, t0 + 32, accB, nB, accA, nA);
      } else if constexpr (b % 2 == 0) {
        step(sQ[b], lam, sub, t0 + 32 * sub, accA, nA, accB, nB);
      } else {
        step(sQ[b], lam, sub, t0 + 32 * sub, accB, nB, accA, nA);
      }
    });
  }
  const int subtiles = KG == 4 ? (nw + 1 - (kg >> 1)) >> 1 : nw;   // this wave's, where it takes one of a tile
  if (KG == 1 || (subtiles & 1) == 0) {
#pragma unroll
    for (int u = 0; u < 32; ++u) exps(accB, nB, u);
  } else {
#pragma unroll
    for (int u = 0; u < 32; ++u) exps(accA, nA, u);
  }
  // the 32 lanes of a half meet; lane (hf, 16 b + i) keeps register i of block b
  float sum = 0.f;
#pragma unroll
  for (int u = 0; u < 32; ++u) {
    float c = col[u >> 4][u & 15];
    c = dpp_add<0x128>(c);   // row_ror 8, 4, 2, 1: the 16 lanes of a row
    c = dpp_add<0x124>(c);
    c = dpp_add<0x122>(c);
    c = dpp_add<0x121>(c);
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(c), __float_as_uint(c), false, false);
    c = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    if (l32 == u) sum = c;
  }
  const int kl = 64 * rg + 32 * (l32 >> 4) + 8 * ((l32 & 15) >> 2) + (l32 & 3) + 4 * hf;   // its key: acc_row
  if constexpr (KG > 1) {
    sCol[kg][kl] = sum;
    tile_barrier();
    if (kg > 0) return;
    double total = (double)sum;   // rounded once, whatever the number of groups
#pragma unroll
    for (int k = 1; k < KG; ++k) total += (double)sCol[k][kl];
    sum = (float)total;
  }
  if (j0 + kl < L) P.S[(size_t)job * L + j0 + kl] = sum * (1.f / (float)G);
}

template <int NRT, int G>
void launch_rows(const PrefillLaunch& P, int n_full, hipStream_t st) {
  constexpr int kPos = RowTiles<NRT, G>::kPositions;
  const int64_t items = (int64_t)n_full * ((P.seq_len + kPos - 1) / kPos);
  fullspan_rows_kernel<NRT, G><<<(unsigned)items, 256, 0, st>>>(P, causal_rows_by_job(items, P.seq_len, P.seq_len));
}

template <int G>
int launch_group(const PrefillLaunch& P, int n_full, hipStream_t st) {
  const int L = P.seq_len;
  bool small = G <= 4 && causal_rows_small(n_full, (int64_t)G * L);
  if constexpr (G <= 4) {
    if (small) launch_rows<4, G>(P, n_full, st);
  }
  if (!small) launch_rows<8, G>(P, n_full, st);
  // Key groups: every query tile a workgroup brings in serves 256, 128 or 64 keys, so as many as leave enough
  // workgroups for an even end.  In blocks of 256 keys: 1024 of them 2045 us a call against 2160 with 128 keys,
  // 576 310 against 310 at L = 1500, 512 1130 against 1005.  64 keys, four waves on a pair of tiles, have the
  // shortest chain of tiles (one job of 840 keys at four heads 54 us against 82 with 128 keys); they are the faster ones up
  // to 128 such blocks at one head a group (192: 52 against 51 us; 288: 78, 72), 256 at two (75, 78; 384: 135, 132) and
  // about 320 from four on (288: 171, 181; 384: 136, 142 at L = 840 and 214, 211 at L = 1500).
  auto blocks = [&](int keys) { return (unsigned)(n_full * ((L + keys - 1) / keys)); };
  if (blocks(256) >= 768) fullspan_cols_kernel<G, 1><<<blocks(256), 256, 0, st>>>(P);
  else if (blocks(256) > (G == 1 ? 128 : G == 2 ? 256 : 320)) fullspan_cols_kernel<G, 2><<<blocks(128), 256, 0, st>>>(P);
  else fullspan_cols_kernel<G, 4><<<blocks(64), 256, 0, st>>>(P);
  return (int)hipGetLastError();
}

}  // namespace

int launch_fullspan(const PrefillLaunch& P, void* stream) {
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int n_full = P.batch * P.n_full * P.n_kv_heads;
  if (n_full <= 0) return 0;
  switch (P.group) {
    case 1: return launch_group<1>(P, n_full, st);
    case 2: return launch_group<2>(P, n_full, st);
    case 4: return launch_group<4>(P, n_full, st);
    case 8: return launch_group<8>(P, n_full, st);
    default: return (int)hipErrorInvalidValue;
  }
}

}  // namespace rkv
