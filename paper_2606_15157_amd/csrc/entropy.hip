// Attention-entropy layer score for capacity allocation (Section 3.3) on gfx950.
//
// H_l is the mean, over sequences, query heads and profiled query positions, of the Shannon
// entropy (nats) of each query's causal attention row: the softmax of q_t . k_j / sqrt(d) over
// keys j = 0..t, query head hq reading KV head hq / G.
//
// entropy_rows_kernel: one workgroup per (layer, sequence, KV head, block of query positions), the row
// pass of causal_rows.h over 128 or 256 query rows of the group.  Per row it takes Z = sum e and
// T = sum e x over the row's keys, e = exp2(x), and
//   H = -sum p ln p = ln 2 (log2 Z - T / Z).
// Bound: 20 cycles of VALU issue per 64 logits beside 16 of the matrix pipe.  256 jobs of 4096 queries and four
// heads: 2.3 ms (3.4 with 16x16x32 MFMA, 32 rows a wave), 2.2 TFLOP of causal logits; the last 515 queries of
// 9001, 128 jobs of two heads: 0.37 ms (0.70).
// A non-finite row is written as it is and reported by the averaging kernel.
// Each workgroup also leaves the double-precision sum of its rows; entropy_mean_kernel (one
// workgroup per layer) adds those in a fixed order.
#include <hip/hip_runtime.h>

#include <math.h>

#include "causal_rows.h"

namespace rkv {
namespace {

template <int NRT, int G>
__global__ __launch_bounds__(256, 2) void entropy_rows_kernel(const EntropyLaunch E, int by_job) {
  constexpr int R = 32 * NRT, PB = RowTiles<NRT, G>::PB, kPos = RowTiles<NRT, G>::kPositions;
  __shared__ CausalRowsLds<NRT> sm;
  __shared__ double sPart[4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int L = E.seq_len, n_q = E.n_q, Hq = E.n_q_heads, Hkv = E.n_kv_heads;
  const int nqb = (n_q + kPos - 1) / kPos;
  const JobItem it = job_item(blockIdx.x, E.n_layers * E.batch * Hkv, nqb, by_job != 0);
  const int qb = nqb - 1 - it.item, i0 = qb * kPos;   // the longest rows first
  const int h = it.job % Hkv, lb = it.job / Hkv, b = lb % E.batch, layer = lb / E.batch;
  const uint16_t* qgroup = E.q[layer] + (size_t)(b * Hq + h * G) * n_q * kHeadDim;
  const uint16_t* khead = E.k[layer] + (size_t)(b * Hkv + h) * L * kHeadDim;
  if (blockIdx.x == 0 && tid == 0 && E.first_group) E.status[0] = 0u;   // once per call: later launches OR into it

  causal_rows<NRT, G, true>(qgroup, n_q, khead, L, i0, E.scale_log2, sm);
  // one thread per row; the workgroup's partial sum in a fixed order (lanes, then waves)
  double part = 0.0;
  if (tid < R) {
    double z = 0.0, t = 0.0;
#pragma unroll
    for (int k = 0; k < CausalRowsLds<NRT>::KG; ++k) {
      z += sm.z[k][tid];
      t += sm.t[k][tid];
    }
    const int rt = tid >> 5, i = i0 + 32 * (rt % PB) + (tid & 31), hq = h * G + rt / PB;
    if (i < n_q) {
      // the logarithm of the mantissa: single precision leaves 3e-8 there, 2e-7 in the logarithm of z
      int ex;
      const float lg = __builtin_log2f((float)frexp(z, &ex));
      const float H = (float)(0.6931471805599453 * ((double)ex + (double)lg - t / z));
      E.rows[((size_t)lb * Hq + hq) * n_q + i] = H;
      part = (double)H;
    }
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) part += __shfl_xor(part, o);
  if (lane == 0) sPart[tid >> 6] = part;
  __syncthreads();
  if (tid == 0) E.partial[(size_t)it.job * nqb + qb] = (sPart[0] + sPart[1]) + (sPart[2] + sPart[3]);
}

__global__ __launch_bounds__(256) void entropy_mean_kernel(const EntropyLaunch E, int nb) {
  __shared__ double sSum[256];
  __shared__ int sBad;
  const int tid = threadIdx.x, layer = blockIdx.x;
  const size_t n = (size_t)E.batch * E.n_q_heads * E.n_q;
  const double* part = E.partial + (size_t)layer * nb;
  if (tid == 0) sBad = 0;
  __syncthreads();
  double s = 0.0;
  for (int r = tid; r < nb; r += 256) s += part[r];
  // a non-finite row makes its block's partial sum non-finite
  if (!(fabs(s) < __builtin_inf())) sBad = 1;
  sSum[tid] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (tid < o) sSum[tid] += sSum[tid + o];
    __syncthreads();
  }
  if (tid == 0) {
    E.h[layer] = (float)(sSum[0] / (double)n);
    if (sBad) atomicOr(E.status, 1u);
  }
}

template <int NRT, int G>
int launch_rows(const EntropyLaunch& E, hipStream_t st) {
  constexpr int kPos = RowTiles<NRT, G>::kPositions;
  const int nqb = (E.n_q + kPos - 1) / kPos, jobs = E.batch * E.n_kv_heads;
  const int64_t items = (int64_t)E.n_layers * jobs * nqb;
  entropy_rows_kernel<NRT, G><<<(unsigned)items, 256, 0, st>>>(E, causal_rows_by_job(items, E.n_q, E.seq_len));
  entropy_mean_kernel<<<E.n_layers, 256, 0, st>>>(E, jobs * nqb);   // nb row blocks per layer
  return (int)hipGetLastError();
}

template <int G>
int launch_group(const EntropyLaunch& E, hipStream_t st) {
  if constexpr (G <= 4) {
    if (causal_rows_small(E.n_layers * E.batch * E.n_kv_heads, E.n_q * G)) return launch_rows<4, G>(E, st);
  }
  return launch_rows<8, G>(E, st);
}

}  // namespace

int launch_entropy(const EntropyLaunch& E, void* stream) {
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  switch (E.n_q_heads / E.n_kv_heads) {
    case 1: return launch_group<1>(E, st);
    case 2: return launch_group<2>(E, st);
    case 4: return launch_group<4>(E, st);
    case 8: return launch_group<8>(E, st);
    default: return (int)hipErrorInvalidValue;
  }
}

}  // namespace rkv
