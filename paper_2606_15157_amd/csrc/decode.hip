// Decode-phase cache update for gfx950: one workgroup per (layer, sequence, KV head).
//
// H2O: the new key joins the C cached keys; every query head of the group scores the C+1
// entries (bf16 dot products accumulated in fp32), takes a softmax, and the group mean of the
// probabilities is added to each entry's fp32 accumulated score.  Among entries outside the
// protected recent window the smallest accumulated score (ties: smallest position) is
// evicted and the new token takes its slot.  TOVA: the same probabilities; an entry's score is
// their group mean at this step alone, every entry (the new one included) is a candidate, and
// the smallest score is evicted (ties: smallest position).  StreamingLLM: the oldest non-sink
// slot is replaced.  Keys are read with 16 lanes per 256-byte row (16 bytes each), so one
// wave's load instruction reads four whole rows.
#include <hip/hip_runtime.h>

#include "rkv_internal.h"

namespace rkv {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x2 as_bf16x2(uint32_t v) { return __builtin_bit_cast(bf16x2, v); }

// Wave reductions by DPP: rotations inside each 16-lane row (every lane of a row ends with the
// row's value), then the four rows' values read from lanes 0, 16, 32 and 48 and combined in that
// order (a fixed order: the sums are reproducible).
template <int CTRL>
__device__ __forceinline__ float dppf(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ __forceinline__ uint32_t dppu(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ float rows4(float v, int i) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 16 * i));
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dppf<0x128>(v));   // row_ror:8
  v = fmaxf(v, dppf<0x124>(v));   // row_ror:4
  v = fmaxf(v, dppf<0x122>(v));   // row_ror:2
  v = fmaxf(v, dppf<0x121>(v));   // row_ror:1
  return fmaxf(fmaxf(rows4(v, 0), rows4(v, 1)), fmaxf(rows4(v, 2), rows4(v, 3)));
}
__device__ __forceinline__ float wave_sum(float v) {
  v += dppf<0x128>(v);
  v += dppf<0x124>(v);
  v += dppf<0x122>(v);
  v += dppf<0x121>(v);
  return (rows4(v, 0) + rows4(v, 1)) + (rows4(v, 2) + rows4(v, 3));
}
// minimum of a 64-bit key (compared as (high word, low word))
template <int CTRL>
__device__ __forceinline__ void min_step(uint32_t& hi, uint32_t& lo) {
  const uint32_t oh = dppu<CTRL>(hi), ol = dppu<CTRL>(lo);
  const bool take = oh < hi || (oh == hi && ol < lo);
  hi = take ? oh : hi;
  lo = take ? ol : lo;
}
__device__ __forceinline__ uint64_t wave_min_u64(uint64_t v) {
  uint32_t hi = (uint32_t)(v >> 32), lo = (uint32_t)v;
  min_step<0x128>(hi, lo);
  min_step<0x124>(hi, lo);
  min_step<0x122>(hi, lo);
  min_step<0x121>(hi, lo);
  uint64_t r = ~0ull;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint64_t x = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, 16 * i) << 32) |
                       (uint32_t)__builtin_amdgcn_readlane((int)lo, 16 * i);
    r = x < r ? x : r;
  }
  return r;
}

template <int NW>
__device__ __forceinline__ uint64_t block_reduce_min_u64(uint64_t v, uint64_t* sh) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  v = wave_min_u64(v);
  if (lane == 0) sh[wv] = v;
  __syncthreads();
  uint64_t r = sh[0];
#pragma unroll
  for (int i = 1; i < NW; ++i) r = sh[i] < r ? sh[i] : r;
  __syncthreads();
  return r;
}

// Block-wide max / sum of G values at once (each value: its waves' results in wave order).
template <int G, int NW>
__device__ __forceinline__ void block_reduce_max_v(float (&v)[G], float* sh) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    v[g] = wave_max(v[g]);
    if (lane == 0) sh[wv * G + g] = v[g];
  }
  __syncthreads();
#pragma unroll
  for (int g = 0; g < G; ++g) {
    float r = sh[g];
#pragma unroll
    for (int i = 1; i < NW; ++i) r = fmaxf(r, sh[i * G + g]);
    v[g] = r;
  }
  __syncthreads();
}
template <int G, int NW>
__device__ __forceinline__ void block_reduce_sum_v(float (&v)[G], float* sh) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    v[g] = wave_sum(v[g]);
    if (lane == 0) sh[wv * G + g] = v[g];
  }
  __syncthreads();
#pragma unroll
  for (int g = 0; g < G; ++g) {
    float r = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) r += sh[i * G + g];
    v[g] = r;
  }
  __syncthreads();
}

template <int G, int NT>
__global__ __launch_bounds__(NT) void decode_kernel(const DecodeLaunch D) {
  constexpr int NW = NT / 64;
  extern __shared__ float sDyn[];
  __shared__ float shf[NW * 8];
  __shared__ uint64_t shu[NW];
  const int tid = threadIdx.x;
  const int Hkv = D.n_kv_heads, B = D.batch;
  const int item = blockIdx.x;
  const int h = item % Hkv, s = (item / Hkv) % B, li = item / (Hkv * B);
  const DecodeLayer& ly = D.layer[li];
  const int C = ly.capacity;
  const int p = D.position;
  const size_t bh = (size_t)s * Hkv + h;
  int32_t* pos = ly.pos + bh * C;
  float* acc = ly.acc ? ly.acc + bh * C : nullptr;   // H2O layers only
  uint16_t* kc = ly.k_cache + bh * C * kHeadDim;
  uint16_t* vc = ly.v_cache + bh * C * kHeadDim;
  const uint16_t* knew = ly.k + bh * kHeadDim;
  const uint16_t* vnew = ly.v + bh * kHeadDim;

  uint64_t best = ~0ull;
  int victim = -1;
  if (ly.rule == RKV_STREAMING) {
    for (int e = tid; e < C; e += NT) {
      const int ps = pos[e];
      if (ps >= D.n_sink) {
        const uint64_t key = ((uint64_t)(uint32_t)ps << 32) | (uint32_t)e;
        best = key < best ? key : best;
      }
    }
    best = block_reduce_min_u64<NW>(best, shu);
    victim = best == ~0ull ? -1 : (int)(uint32_t)(best & 0xffffffffu);
  } else {
    float* sZ = sDyn;                      // [G][C+1] logits, then probabilities
    float* sAcc = sDyn + (size_t)G * (C + 1);  // [C+1] updated accumulated scores
    // 16 lanes per entry: lane c (= tid % 16) takes the 16-byte chunk c of the head dimension, so
    // a wave's load instruction reads four whole 256-byte rows; lanes hold chunk c of every
    // query head.  An iteration covers NT / 4 entries, entry base + tid / 16 + j NT / 16 for j = 0..3.
    const int c16 = tid & 15, rsub = tid >> 4;
    u32x4 qr[G];
#pragma unroll
    for (int g = 0; g < G; ++g)
      qr[g] = reinterpret_cast<const u32x4*>(ly.q + ((size_t)s * D.n_q_heads + h * G + g) * kHeadDim)[c16];
    constexpr int kBlk = NT / 4;   // entries per block
    // two blocks of key rows in flight: block b + 1's loads are outstanding while block b's dot
    // products run, and block b + 2's are issued right after them (two register sets,
    // alternating).  Every load is unconditional (entries past the end read the new token's row,
    // which the cache serves), so the compiler's waits leave the other block in flight.
    auto load_rows = [&](int base, u32x4 (&kv)[4]) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int e = base + rsub + NT / 16 * j;
        const uint16_t* kr = e < C ? kc + (size_t)e * kHeadDim : knew;
        kv[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kr) + c16);
      }
    };
    float mx[G];
#pragma unroll
    for (int g = 0; g < G; ++g) mx[g] = -__builtin_inff();
    // dot products of the block at base (rows in kv), summed over the 16 lanes of each entry
    // (one DPP row, every lane gets the sum); one lane writes each logit to LDS
    auto process = [&](int base, const u32x4 (&kv)[4]) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int e = base + rsub + NT / 16 * j;
#pragma unroll
        for (int g = 0; g < G; ++g) {
          float d = 0.f;
#pragma unroll
          for (int u = 0; u < 4; ++u) d = __builtin_amdgcn_fdot2_f32_bf16(as_bf16x2(kv[j][u]), as_bf16x2(qr[g][u]), d, false);
          d += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, d), 0x128, 0xf, 0xf, false));
          d += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, d), 0x124, 0xf, 0xf, false));
          d += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, d), 0x122, 0xf, 0xf, false));
          d += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, d), 0x121, 0xf, 0xf, false));
          if (e <= C) {
            mx[g] = fmaxf(mx[g], d);
            if (c16 == ((j * G + g) & 15)) sZ[g * (C + 1) + e] = d;
          }
        }
      }
    };
    u32x4 ka[4], kb[4];
    load_rows(0, ka);
    load_rows(kBlk, kb);
    for (int base = 0; base <= C; base += 2 * kBlk) {
      process(base, ka);
      load_rows(base + 2 * kBlk, ka);
      process(base + kBlk, kb);
      load_rows(base + 3 * kBlk, kb);
    }
    // H2O: candidates have position <= p - r and the score accumulates; TOVA: every entry is a
    // candidate and the score is this step's alone
    const bool tova = ly.rule == RKV_TOVA;
    const int limit = tova ? p : p - ly.recent;
    // positions and accumulated scores of entries tid + NT k (k < kDecPre), requested now so
    // that they arrive during the reductions and the exponential pass (the key registers are
    // free here); entries past those are read when visited
    constexpr int kDecPre = NT == 256 ? 4 : 2;
    int pre_pos[kDecPre];
    float pre_acc[kDecPre];
#pragma unroll
    for (int k = 0; k < kDecPre; ++k) {
      const int e = tid + NT * k;
      pre_pos[k] = e < C ? pos[e] : p;
      pre_acc[k] = e < C && !tova ? acc[e] : 0.f;
    }
    // every head's maximum and row sum in one pass over the logits, two block reductions
    const float sl2 = D.scale_log2;
    block_reduce_max_v<G, NW>(mx, shf);   // its first barrier also publishes the logits in LDS
    float sm[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      mx[g] *= sl2;
      sm[g] = 0.f;
    }
    for (int e = tid; e <= C; e += NT) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float x = __builtin_amdgcn_exp2f(fmaf(sZ[g * (C + 1) + e], sl2, -mx[g]));
        sZ[g * (C + 1) + e] = x;
        sm[g] += x;
      }
    }
    block_reduce_sum_v<G, NW>(sm, shf);
    float inv[G];
#pragma unroll
    for (int g = 0; g < G; ++g) inv[g] = 1.0f / sm[g];
    auto visit = [&](int e, float acc_e, int ps) {
      float pm = 0.f;
#pragma unroll
      for (int g = 0; g < G; ++g) pm += sZ[g * (C + 1) + e] * inv[g];
      pm = pm / (float)G;
      const float a = acc_e + pm;
      sAcc[e] = a;
      if (ps <= limit) {
        const uint64_t key = ((uint64_t)__float_as_uint(a) << 32) | (uint32_t)ps;
        best = key < best ? key : best;
      }
    };
#pragma unroll
    for (int k = 0; k < kDecPre; ++k)
      if (tid + NT * k <= C) visit(tid + NT * k, pre_acc[k], pre_pos[k]);
    for (int e = tid + NT * kDecPre; e <= C; e += NT)
      visit(e, e < C && !tova ? acc[e] : 0.f, e < C ? pos[e] : p);
    best = block_reduce_min_u64<NW>(best, shu);
    const int vpos = (int)(uint32_t)(best & 0xffffffffu);
    // slot holding the winning position (positions are distinct); C = the new token
    __shared__ int sVictim;
    if (tid == 0) sVictim = -1;
    __syncthreads();
    if (best != ~0ull) {
#pragma unroll
      for (int k = 0; k < kDecPre; ++k)
        if (tid + NT * k <= C && pre_pos[k] == vpos) sVictim = tid + NT * k;
      for (int e = tid + NT * kDecPre; e <= C; e += NT) {
        const int ps = e < C ? pos[e] : p;
        if (ps == vpos) sVictim = e;
      }
    }
    __syncthreads();
    victim = sVictim;
    if (victim == C) victim = -1;
    if (!tova)
      for (int e = tid; e < C; e += NT) acc[e] = (e == victim) ? sAcc[C] : sAcc[e];
  }
  // the new token takes the victim's slot
  if (victim >= 0) {
    if (tid < 16) {
      reinterpret_cast<u32x4*>(kc + (size_t)victim * kHeadDim)[tid] = reinterpret_cast<const u32x4*>(knew)[tid];
    } else if (tid < 32) {
      reinterpret_cast<u32x4*>(vc + (size_t)victim * kHeadDim)[tid - 16] = reinterpret_cast<const u32x4*>(vnew)[tid - 16];
    } else if (tid == 32) {
      pos[victim] = p;
    }
  }
  if (tid == 0 && ly.victim) ly.victim[bh] = victim;
}

template <int G, int NT>
int launch_decode_kernel(const DecodeLaunch& D, unsigned grid, size_t lds, hipStream_t st) {
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(decode_kernel<G, NT>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
    if (e != hipSuccess) return (int)e;
    attr_set = true;
  }
  profile_mark(kStageDecode, false, st);
  decode_kernel<G, NT><<<grid, NT, lds, st>>>(D);
  profile_mark(kStageDecode, true, st);
  return (int)hipGetLastError();
}

template <int G>
int launch_decode_group(const DecodeLaunch& D, int max_capacity, hipStream_t st) {
  const unsigned grid = (unsigned)(D.n_layers * D.batch * D.n_kv_heads);
  const size_t lds = sizeof(float) * (size_t)(G + 1) * (max_capacity + 1);
  // Twice the waves a workgroup, so twice the key rows in flight, where the workgroups leave a CU few of them:
  // one workgroup per CU (256 of 512 entries: 16.0 -> 13.4 us, of 2048: 44 -> 31; below 128 entries a second
  // block of rows is empty: 64: 7.1 -> 8.0), or few by their LDS with more of them waiting.  With eight heads a group that
  // is three (2048 workgroups of 1500 entries: 274 -> 216 us, of 2048 376 -> 294): the registers leave 20 waves a
  // CU, so four of 512 threads do not fit where four of 256 do (of 1000 entries 141 -> 152, 6144 of them 384 ->
  // 434).  With fewer heads it is four (2048 of 4000 entries at four heads 430 -> 379, of 2048 203 -> 197, of 3000 at
  // two 281 -> 278; five: 1500 at four 143.7 -> 143.9, 4000 at one 351 -> 359).  Otherwise the smaller ones end more
  // evenly (512 of 512 entries: 19.7 against 20.8; 16384 of 1024: 716 against 726).  Four times the waves
  // measured slower everywhere (256 of 512: 16.1, 16384 of 1024: 1233).
  const size_t by_lds = 160 * 1024 / lds;
  const bool wide = grid <= 256 ? max_capacity >= 128 : by_lds <= (G == 8 ? 3 : 4) && grid > 256 * by_lds;
  return wide ? launch_decode_kernel<G, 512>(D, grid, lds, st) : launch_decode_kernel<G, 256>(D, grid, lds, st);
}

}  // namespace

int launch_decode(const DecodeLaunch& D, int max_capacity, void* stream) {
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  switch (D.group) {
    case 1: return launch_decode_group<1>(D, max_capacity, st);
    case 2: return launch_decode_group<2>(D, max_capacity, st);
    case 4: return launch_decode_group<4>(D, max_capacity, st);
    case 8: return launch_decode_group<8>(D, max_capacity, st);
    default: return (int)hipErrorInvalidValue;
  }
}

}  // namespace rkv
