// Log-sum-exp merge of split rows: the float32 partials that decode units wrote for
// the pieces of one (sequence, KV head) row become its bf16 output and float32 LSE.
//
// One 256-thread block per query head of a split row: up to 16 groups of 16 threads, thread t
// of a group channels 8 t .. + 7.  Group k folds splits k, k + groups, ... four at a time
// (all loads of a batch in flight) with a running maximum, so up to 64 splits take one round
// of loads; the groups' (max, sum, accumulator) then combine by lane shuffles within a wave
// and through LDS across the four waves, in a fixed order.  With M = max_j lse_j (base 2):
// lse = M + log2(sum_j 2^(lse_j - M)), o = sum_j 2^(lse_j - lse) o_j; empty splits
// (lse_j = -inf) add nothing.  Bound by latency (record, one round of loads, combine, store),
// so splits are spread over the block rather than looped over, and a row of at most 16 splits
// uses one wave, one of at most four a single group.  Kernel time for two rows of two splits
// (8 heads): 2.7 us with a block per row whose threads looped over the splits, 3.2 with 16
// groups for every row, 2.5 now; for the 8 rows of a 40,960-token request (40 heads) 5.1 us
// in 64 splits, and in the 32 that are launched since 4.6 and 4.5 us.
#include <algorithm>
#include <cmath>

#include "internal.h"

namespace libra {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;
constexpr int kBatch = 8;
constexpr float kLn2 = 0.6931471805599453f;

// Two floats to bf16 (round to nearest even) in one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

struct MergeArgs {
  const int32_t* merges;
  const float* part_o;
  const float* part_lse;
  uint16_t* out;
  float* lse;
  int hq;
  int group;
};

__global__ __launch_bounds__(kThreads) void merge_kernel(MergeArgs A) {
  constexpr int kGroups = kThreads / 16, kWaves = kThreads / 64, kRowBatch = 4;
  __shared__ float red_m[kWaves][16];
  __shared__ float red_w[kWaves][16];
  __shared__ __align__(16) float red_acc[kWaves][16][12];  // padded row

  const int G = A.group;
  const int32_t* m = A.merges + size_t(blockIdx.x) * kMergeInts;
  const int h = blockIdx.y;
  const int g = m[M_G], n = m[M_N], part = m[M_PART], row = m[M_ROW];
  const int tid = threadIdx.x, t = tid & 15, grp = tid >> 4;
  // Few splits: as many groups as one batch of loads each needs, and only the rounds of the
  // combine that these take.  Uniform over the block.
  const int groups = n <= kRowBatch ? 1 : n <= kRowBatch * 4 ? 4 : kGroups;
  if (grp >= groups) return;

  float M = -INFINITY, wsum = 0.f;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // Folds (Mk, wk, xk) into the running triple.
  auto fold = [&](float Mk, float wk, const float (&xk)[8]) {
    const float Mn = fmaxf(M, Mk);
    const float a = Mn == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - Mn);
    const float b = Mn == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(Mk - Mn);
    wsum = wsum * a + wk * b;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = acc[i] * a + xk[i] * b;
    M = Mn;
  };
  for (int j0 = grp; j0 < n; j0 += kRowBatch * groups) {
    float lj[kRowBatch];
    f32x4 x0[kRowBatch], x1[kRowBatch];
#pragma unroll
    for (int jj = 0; jj < kRowBatch; ++jj) {
      const int j = j0 + jj * groups;
      lj[jj] = -INFINITY;
      x0[jj] = x1[jj] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (j < n) {
        const size_t slot = size_t(part + j) * G + h;
        lj[jj] = A.part_lse[slot];
        const float* po = A.part_o + slot * kDim + 8 * t;
        x0[jj] = *reinterpret_cast<const f32x4*>(po);
        x1[jj] = *reinterpret_cast<const f32x4*>(po + 4);
      }
    }
    float Mc = M;
#pragma unroll
    for (int jj = 0; jj < kRowBatch; ++jj) Mc = fmaxf(Mc, lj[jj]);
    if (Mc == -INFINITY) continue;
    const float r = __builtin_amdgcn_exp2f(M - Mc);  // 0 while M = -inf
    wsum *= r;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] *= r;
#pragma unroll
    for (int jj = 0; jj < kRowBatch; ++jj) {
      const float w = __builtin_amdgcn_exp2f(lj[jj] - Mc);  // 0 for empty or absent splits
      wsum += w;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[i] += w * x0[jj][i];
        acc[4 + i] += w * x1[jj][i];
      }
    }
    M = Mc;
  }
  if (groups > 1) {
#pragma unroll
    for (int d = 16; d < 64; d *= 2) {
      float x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = __shfl_xor(acc[i], d);
      const float Mk = __shfl_xor(M, d), wk = __shfl_xor(wsum, d);
      fold(Mk, wk, x);
    }
  }
  if (groups > 4) {
    const int wave = tid >> 6;
    if ((tid & 63) < 16) {
      red_m[wave][t] = M;
      red_w[wave][t] = wsum;
#pragma unroll
      for (int i = 0; i < 8; ++i) red_acc[wave][t][i] = acc[i];
    }
    __syncthreads();
    if (tid < 16) {
#pragma unroll
      for (int k = 1; k < kWaves; ++k) {
        float x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = red_acc[k][t][i];
        fold(red_m[k][t], red_w[k][t], x);
      }
    }
  }
  if (tid >= 16) return;
  const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
  uint4 ov;
  ov.x = pack_bf16x2(acc[0] * inv, acc[1] * inv);
  ov.y = pack_bf16x2(acc[2] * inv, acc[3] * inv);
  ov.z = pack_bf16x2(acc[4] * inv, acc[5] * inv);
  ov.w = pack_bf16x2(acc[6] * inv, acc[7] * inv);
  const size_t out_row = size_t(row) * A.hq + size_t(g) * G + h;
  *reinterpret_cast<uint4*>(A.out + out_row * kDim + 8 * t) = ov;
  if (A.lse && t == 0) A.lse[out_row] = wsum > 0.f ? (M + log2f(wsum)) * kLn2 : -INFINITY;
}

// Log-sum-exp merge of the fine tiles whose keys were split, over kTileRows rows of
// (token, head) pairs each.  A 256-thread block takes two rows: eight groups of 32 threads,
// four to a row, thread t of a group channels 4 t .. + 3.  Group k of a row folds splits k,
// k + 4, ... eight at a time (all loads of a batch in flight), and the groups combine
// through LDS.  Latency-bound: many small blocks and at most ceil(n / 32) dependent rounds
// of loads.  A split without a key of the row (lse_j = -inf) is left out by its weight and
// its partial (which may hold another row's NaN); a NaN lse_j or partial of a split that
// the row sees makes the row NaN, as it does where keys are not split: maxima ignore NaN, so
// no batch or group is skipped by its maximum.
constexpr int kRowGroups = 4;
constexpr int kMergeRows = kThreads / (32 * kRowGroups);

__global__ __launch_bounds__(kThreads) void chunk_merge_kernel(MergeArgs A) {
  __shared__ float red_m[kMergeRows][kRowGroups];
  __shared__ float red_w[kMergeRows][kRowGroups];
  __shared__ __align__(16) f32x4 red_acc[kMergeRows][kRowGroups][32];

  const int32_t* m = A.merges + size_t(blockIdx.x) * kMergeInts;
  const int g = m[CM_GH] & 0xFFFF, first = (m[CM_GH] >> 16) * kTileRows;
  const int n = m[CM_N], part = m[CM_PART];
  const int tid = threadIdx.x, t = tid & 31, grp = (tid >> 5) % kRowGroups;
  const int lr = tid / (32 * kRowGroups);
  const int r = blockIdx.y * kMergeRows + lr;  // row of the workgroup's kTileRows
  const int G = A.group;
  const int tok = m[CM_Q0] + (first + r) / G, head = (first + r) % G;
  const bool ok = tok < m[CM_Q1];

  float M = -INFINITY, wsum = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (ok) {
    for (int j0 = grp; j0 < n; j0 += kBatch * kRowGroups) {
      float lj[kBatch];
      f32x4 x[kBatch];
#pragma unroll
      for (int jj = 0; jj < kBatch; ++jj) {
        const int j = j0 + jj * kRowGroups;
        lj[jj] = -INFINITY;
        x[jj] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (j < n) {
          const size_t row = size_t(part + j) * kTileRows + r;
          lj[jj] = A.part_lse[row];
          x[jj] = *reinterpret_cast<const f32x4*>(A.part_o + row * kDim + 4 * t);
        }
      }
      float Mc = M;
#pragma unroll
      for (int jj = 0; jj < kBatch; ++jj) Mc = fmaxf(Mc, lj[jj]);
      const float s = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - Mc);
      wsum *= s;
      acc *= s;
#pragma unroll
      for (int jj = 0; jj < kBatch; ++jj) {
        if (lj[jj] == -INFINITY) continue;  // empty or absent split
        const float w = __builtin_amdgcn_exp2f(lj[jj] - Mc);
        wsum += w;
        acc += w * x[jj];
      }
      M = Mc;
    }
  }
  if (t == 0) {
    red_m[lr][grp] = M;
    red_w[lr][grp] = wsum;
  }
  red_acc[lr][grp][t] = acc;
  __syncthreads();
  if (grp != 0 || !ok) return;
#pragma unroll
  for (int k = 1; k < kRowGroups; ++k) {
    const float Mk = red_m[lr][k];
    const float Mn = fmaxf(M, Mk);
    const float a = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - Mn);
    const float b = Mk == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(Mk - Mn);
    wsum = wsum * a + red_w[lr][k] * b;
    acc = acc * a + red_acc[lr][k][t] * b;
    M = Mn;
  }
  const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
  const size_t row = size_t(m[CM_ROW0] + tok) * A.hq + size_t(g) * G + head;
  *reinterpret_cast<uint2*>(A.out + row * kDim + 4 * t) =
      make_uint2(pack_bf16x2(acc.x * inv, acc.y * inv), pack_bf16x2(acc.z * inv, acc.w * inv));
  if (A.lse && t == 0) A.lse[row] = wsum > 0.f ? (M + log2f(wsum)) * kLn2 : -INFINITY;
}

}  // namespace

bool merge_launches(const Plan& P) { return P.info.n_merge_groups > 0 || !P.chunk_merges.empty(); }

hipError_t launch_merge(const Plan& P, void* ws, void* out, float* lse, hipStream_t s) {
  const int n = P.info.n_merge_groups;
  char* w = static_cast<char*>(ws);
  MergeArgs A;
  A.merges = reinterpret_cast<const int32_t*>(w + P.off_merges);
  A.part_o = reinterpret_cast<const float*>(w + P.off_part_o);
  A.part_lse = reinterpret_cast<const float*>(w + P.off_part_lse);
  A.out = static_cast<uint16_t*>(out);
  A.lse = lse;
  A.hq = P.num_q_heads;
  A.group = P.group;
  // Blocks (record, head); a grid's dimension holds at most 2^32 - 1 work-items.
  const int32_t* const first = A.merges;
  constexpr int kMost = 1 << 23;
  for (int r0 = 0; r0 < n; r0 += kMost) {
    A.merges = first + size_t(r0) * kMergeInts;
    hipLaunchKernelGGL(merge_kernel, dim3(unsigned(std::min(kMost, n - r0)), unsigned(P.group)),
                       dim3(kThreads), 0, s, A);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (!P.chunk_merges.empty()) {
    A.merges = reinterpret_cast<const int32_t*>(w + P.off_chunk_merges);
    A.part_o = reinterpret_cast<const float*>(w + P.off_chunk_o);
    A.part_lse = reinterpret_cast<const float*>(w + P.off_chunk_lse);
    hipLaunchKernelGGL(chunk_merge_kernel,
                       dim3(unsigned(P.chunk_merges.size() / kMergeInts), kTileRows / kMergeRows),
                       dim3(kThreads), 0, s, A);
    return hipGetLastError();
  }
  return hipSuccess;
}

}  // namespace libra
