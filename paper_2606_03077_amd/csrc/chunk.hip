// Causal attention of an appended chunk (e.g. a tool output) over the paged KV cache.
//
// Two forms of one kernel.  The wide form is a 512-thread workgroup (8 waves, two per SIMD,
// one workgroup per CU) per chunk unit (sequence b, KV head g, new tokens [q0, q1)), up to
// 256 query rows.  The narrow form is a 256-thread workgroup (4 waves, two workgroups per
// CU) per fine tile: half of a unit's rows, over the keys that they see or one split of them
// (the plan decides; the rule and its measurements stand in plan.cpp).  Query rows are the
// (token, head) pairs of the G heads sharing KV head g, token-major; wave w owns 32 of them
// as the 32 columns of its matrix products.
// Keys are visited 64 (wide) or 32 (narrow) at a time: a step of four pages, two page
// pairs, or of one pair.  The step's K and V tiles are copied from memory straight into a
// four-stage LDS ring three steps ahead (global_load_lds_dwordx4, 16 bytes per lane, the
// tiles in their stored order, no registers), shared by the waves.  Per page pair and wave,
// on v_mfma_f32_32x32x16_bf16:
//   S^T[32 keys x 32 rows] = K . Q^T: 8 MFMAs over the 128 channels; lane (key m, half
//     h) reads K granule (2 c + h) * 16 + m % 16 of page 2P + m / 16 for channels
//     16 c + 8 h .. + 7, and holds scores of keys 8 (r / 4) + 4 h + r % 4 (r = 0..15)
//     for its row;
//   O^T[128 channels x 32 rows] += V^T . P^T: per page, 4 MFMAs (32-channel blocks) over
//     the page's 16 keys.  A lane's probabilities of one page, keys {4h..4h+3, 8+4h..
//     11+4h} in that order, are its B operand as they come out of the scores; the
//     matching A operand, channel d's values at those keys, is V granule 128 h + d of
//     the stored tile (one 16-byte LDS read; the 32 lanes of one half read 512 contiguous
//     bytes, free of bank conflicts), which is why V tiles are stored in that order.
// Each wave works through a step by page pairs: the pair's K operands for step n + 1
// are read from LDS first, then the pair's probabilities are formed (exps) while they
// land, then step n + 1's scores of the pair (a dependent chain of 8 MFMAs) are issued
// interleaved with the pair's 8 independent PV products.
// Softmax runs online in base 2 against a running maximum that is set exactly on the
// first step and afterwards moved only when needed: the probabilities of a page pair
// are taken against the current maximum, and if any lane's sum of them exceeds 2^kTau
// (which any probability above 2^kTau forces), a wave-wide vote moves the maximum to
// the pair's own, rescales the accumulators and takes them again, before a product uses
// them.  Probabilities therefore stay at most 2^kTau, and the result is exact after the
// final normalisation; no per-step maximum is taken.  Causal masks are applied only on
// steps that reach past the tile's first token.  Row r of the unit is token q0 + r / G,
// head r % G; it sees keys k <= P_b + token.
// Workgroups arrive in per-XCD queues: workgroup w takes tile w / 8 of queue w % 8, so the
// tiles of one (b, g), which read the same keys, run on one XCD and share its L2; each
// queue holds its longest tiles first.
//
// What bounds it: the matrix cores and the softmax's vector work beside them on long tiles
// (wide form 1.21-1.27 PFLOP/s on a 40,960-token prefill; the narrow form is 8% slower
// there, as every 128 rows copy their own K and V), and the work per tile on short ones.
// Skipping the ring's copies past the last key, starting the first copies from scalar page
// ids and storing whole rows through LDS took 32 prompts of 64-2,048 tokens (40/8 heads) as
// whole units from 893 us to 858 us on one card, cache write included; the narrow form takes
// 857 us on them.
#include <cfloat>
#include <cmath>
#include <type_traits>

#include "internal.h"

namespace libra {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kWideWaves = 8;
constexpr int kNarrowWaves = 4;
static_assert(kChunkRows == 32 * kWideWaves, "the plan's tile rows are the wide form's");
static_assert(kTileRows == 32 * kNarrowWaves, "the fine tiles' rows are the narrow form's");
// Pages (16 keys each) per softmax step: one page pair for every four waves, so that each
// wave moves the same two 1 KiB chunks of K and of V per step in either form.
constexpr int step_pages(int waves) { return waves / 2; }
static_assert(step_pages(kWideWaves) * kPage == kChunkStepKeys, "the plan's tile cost counts these steps");
static_assert(step_pages(kNarrowWaves) * kPage == kTileStepKeys, "the plan cuts key ranges at whole steps");
constexpr int kTau = 8;           // lazy-rescale threshold, base-2 logits
constexpr float kSumTau = float(1 << kTau);  // probabilities stay at most 2^kTau
constexpr int kMaxIds = 4096;     // block-table entries staged in LDS (64K keys)
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 x) { return __builtin_bit_cast(bf16x8, x); }
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

struct ChunkArgs {
  const uint16_t* k_cache;
  const uint16_t* v_cache;
  const int32_t* units;
  const int32_t* tiles;
  const int32_t* bt;
  const uint16_t* q;
  uint16_t* out;
  float* lse;
  float* part_o;
  float* part_lse;
  int64_t bt_stride;
  int hkv;
  int hq;
  int group;
  float sl2;
  int form;         // ChunkForm
  int half_tokens;  // tokens that a unit's first half touches
  int32_t xcd_first[kNumXcds];  // each XCD queue's first record and workgroup count
  int32_t xcd_count[kNumXcds];
};

// Row (M index) of element r of a 32x32 accumulator in a lane of half h.
__device__ __forceinline__ constexpr int acc_row(int r, int h) { return 8 * (r / 4) + 4 * h + (r % 4); }

template <int kWaves>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void chunk_kernel(ChunkArgs A) {
  constexpr bool kWide = kWaves == kWideWaves;
  constexpr int kThreads = 64 * kWaves;
  constexpr int kRows = 32 * kWaves;
  constexpr int kStepPages = step_pages(kWaves);
  constexpr int kPairs = kStepPages / 2;
  constexpr int kStepKeys = kStepPages * kPage;
  // K and V stages: [page of the step][256 x uint4], the tiles as stored.  One array per
  // stage: the direct memory-to-LDS copies into one stage then never make the compiler
  // wait before LDS reads of another.
  __shared__ __align__(16) uint4 ldk0[kStepPages][256];
  __shared__ __align__(16) uint4 ldk1[kStepPages][256];
  __shared__ __align__(16) uint4 ldk2[kStepPages][256];
  __shared__ __align__(16) uint4 ldk3[kStepPages][256];
  __shared__ __align__(16) uint4 ldv0[kStepPages][256];
  __shared__ __align__(16) uint4 ldv1[kStepPages][256];
  __shared__ __align__(16) uint4 ldv2[kStepPages][256];
  __shared__ __align__(16) uint4 ldv3[kStepPages][256];
  __shared__ __align__(16) int lds_ids[kMaxIds];
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  using S2 = std::integral_constant<int, 2>;
  using S3 = std::integral_constant<int, 3>;
  auto kst = [&](auto s_tag) -> uint4 (&)[kStepPages][256] {
    constexpr int st = decltype(s_tag)::value & 3;
    if constexpr (st == 0) return ldk0;
    else if constexpr (st == 1) return ldk1;
    else if constexpr (st == 2) return ldk2;
    else return ldk3;
  };
  auto vst = [&](auto s_tag) -> uint4 (&)[kStepPages][256] {
    constexpr int st = decltype(s_tag)::value & 3;
    if constexpr (st == 0) return ldv0;
    else if constexpr (st == 1) return ldv1;
    else if constexpr (st == 2) return ldv2;
    else return ldv3;
  };

  const int xcd = blockIdx.x % kNumXcds;
  const int slot = blockIdx.x / kNumXcds;
  if (slot >= A.xcd_count[xcd]) return;
  const size_t rec = size_t(A.xcd_first[xcd] + slot);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int col = lane & 31, hh = lane >> 5;  // accumulator column (tile row), lane half
  const int G = A.group;

  // The workgroup's rows are r_first .. r_first + kRows - 1 of the (token, head) rows of
  // tokens [q0, q1), its keys [kv0, kv1).  The wide form takes a plan unit, the narrow one
  // half of a unit's rows: over the keys that they see, straight from the unit's record, or
  // over one split of them, from a fine tile's.
  int b, g, q0, q1, row0, prior, kv0, kv1, r_first, nsplit, part;
  if (kWide || A.form != kFineTiles) {
    size_t unit = rec;
    int half = 0;
    if (!kWide && A.form == kBothHalves) {
      unit = size_t(A.xcd_first[xcd] + (slot >> 1)), half = slot & 1;
    } else if (!kWide && A.form == kListedHalves) {
      unit = size_t(A.tiles[rec] >> 1), half = A.tiles[rec] & 1;
    }
    const int32_t* u = A.units + unit * kUnitInts;
    b = u[U_B], g = u[U_G], q0 = u[U_Q0], q1 = u[U_Q1], row0 = u[U_ROW0], prior = u[U_PRIOR];
    kv0 = 0, kv1 = u[U_KV1], r_first = half * kRows, nsplit = 1, part = 0;
    if (!kWide && !half) kv1 = min(kv1, prior + q0 + A.half_tokens);
  } else {
    const int32_t* u = A.tiles + rec * kTileInts;
    b = u[T_B], g = u[T_GH] & 0xFFFF, q0 = u[T_Q0], q1 = u[T_Q1], row0 = u[T_ROW0];
    prior = u[T_PRIOR], kv0 = u[T_KV0], kv1 = u[T_KV1], r_first = (u[T_GH] >> 16) * kRows;
    nsplit = u[T_NSPLIT], part = u[T_PART];
  }
  const int npages = (kv1 - kv0 + kPage - 1) / kPage;  // kv0 is a multiple of the step
  const int nsteps = (npages + kStepPages - 1) / kStepPages;
  const int last = nsteps - 1;
  const int32_t* btrow = A.bt + int64_t(b) * A.bt_stride + kv0 / kPage;
  // Page ids of this wave's chunks of the first three steps, by scalar loads: the first
  // copies then wait for neither the staged id row nor its barrier.
  const int wpage = wave >> 1;
  int first_id[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) first_id[i] = btrow[min(i * kStepPages + wpage, npages - 1)];

  // Tile row of this lane's column: r = r_first + 32 wave + col; token q0 + r / G,
  // head r % G.
  const int r_tile = r_first + 32 * wave + col;
  const int t_tok = q0 + r_tile / G;
  const int head = r_tile % G;
  const bool ok = t_tok < q1;
  const int lim = ok ? prior + t_tok : -1;
  // Q operand of MFMA c (channels 16 c .. 16 c + 15): lane (col, hh) holds channels
  // 16 c + 8 hh .. + 7 of its row.
  bf16x8 qop[8];
  {
    const uint4* qrow = reinterpret_cast<const uint4*>(
        A.q + (size_t(row0 + (ok ? t_tok : 0)) * A.hq + size_t(g) * G + head) * kDim);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      uint4 v = make_uint4(0, 0, 0, 0);
      if (ok) v = qrow[2 * c + hh];
      qop[c] = as_bf16x8(v);
    }
  }

  float m = -INFINITY, l = 0.f;
  f32x16 acc[4];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[cb][r] = 0.f;

  const uint32_t page_bytes = uint32_t(A.hkv) * kTileBytes;
  const int first_tok = prior + q0 + r_first / G;
  const int mask_key0 = min(first_tok - (kStepPages * kPage - 1), kv1 - kStepPages * kPage);

  const char* k_lane = reinterpret_cast<const char*>(A.k_cache) + size_t(g) * kTileBytes +
                       size_t(lane) * 16;
  const char* v_lane = reinterpret_cast<const char*>(A.v_cache) + size_t(g) * kTileBytes +
                       size_t(lane) * 16;
  // K or V of a step straight into an LDS stage: wave w moves 1 KiB chunks 2 w and 2 w + 1
  // of the step's tiles (16 B per lane at the chunk's LDS base + 16 lane, the tile as
  // stored).  Both chunks lie in page w / 2 of the step, so a wave needs one page id: from
  // the staged row (a broadcast LDS read), or from global memory past it (uniform and
  // rare).  Pages past the end re-read the last page (the id row is padded with it); their
  // keys are >= kv1, so they are masked and their V zeroed.  The wave index is made scalar,
  // so the page, the LDS targets and the byte offsets are scalar arithmetic.  Two
  // vector-memory operations per wave and call, in a fixed order; the waits count them.
  auto tile_off = [&](int id) -> uint64_t { return uint64_t(uint32_t(id)) * page_bytes; };
  auto page_off = [&](int step) -> uint64_t {
    const int p = step * kStepPages + wpage;
    return tile_off(p < kMaxIds ? __builtin_amdgcn_readfirstlane(lds_ids[p])
                                : __builtin_amdgcn_readfirstlane(btrow[min(p, npages - 1)]));
  };
  auto copy_tile = [&](const char* src, uint4 (&dst)[kStepPages][256], uint64_t off) {
#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2) {
      const int i = (2 * wave + c2) & 3;
      const uint32_t d = uint32_t(reinterpret_cast<uintptr_t>(&dst[wpage][i * 64]));
      const char* s = src + (off + i * 1024);
      asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off"
                   :
                   : "s"(d), "v"(s)
                   : "memory", "m0");
    }
  };
  copy_tile(k_lane, kst(S0{}), tile_off(first_id[0]));
  copy_tile(v_lane, vst(S0{}), tile_off(first_id[0]));
  if (last > 0) {
    copy_tile(k_lane, kst(S1{}), tile_off(first_id[1]));
    copy_tile(v_lane, vst(S1{}), tile_off(first_id[1]));
  }
  if (last > 1) {
    copy_tile(k_lane, kst(S2{}), tile_off(first_id[2]));
    copy_tile(v_lane, vst(S2{}), tile_off(first_id[2]));
  }
  // Stage the later steps' page ids once (padded to whole steps with the last id), so that
  // each later copy is one dependent load, not two; four loads in flight per thread.
  const int nids = min(nsteps * kStepPages, kMaxIds);
  for (int i0 = 3 * kStepPages + tid; i0 < nids; i0 += 4 * kThreads) {
    int v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = btrow[min(i0 + j * kThreads, npages - 1)];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (i0 + j * kThreads < nids) lds_ids[i0 + j * kThreads] = v[j];
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  // Scores S^T (32 keys of page pair P x 32 rows) from K stage: K operand of MFMA c,
  // lane (key m, hh): slot m % 16 of page 2P + m / 16, channels 16 c + 8 hh .. + 7, the
  // K granule (2 c + hh) * 16 + slot.
  auto qk_pair = [&](auto stage_tag, int P, f32x16& s) {
    f32x16 a;
#pragma unroll
    for (int r = 0; r < 16; ++r) a[r] = 0.f;
    const int j = 2 * P + (col >> 4);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const uint4 kr = kst(stage_tag)[j][(2 * c + hh) * 16 + (col & 15)];
      a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kr), qop[c], a, 0, 0, 0);
    }
    s = a;
  };

  // Causal / length mask of step n; on the first step (exact) also the running maximum
  // (later steps check their probabilities instead, in pair()).  While no finite score has
  // come (a row without keys here, or whose first keys score -inf), the offset is the
  // largest float: scores of -inf still give 0, and the first finite one gives infinity,
  // which makes pair() set the maximum.
  auto prepare = [&](int key0, f32x16 (&s)[kPairs], float& neg_m, bool exact) {
    if (key0 > mask_key0) {
#pragma unroll
      for (int P = 0; P < kPairs; ++P)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (key0 + 32 * P + acc_row(r, hh) > lim) s[P][r] = -INFINITY;
    }
    if (exact) {
      float mloc = -INFINITY;
#pragma unroll
      for (int P = 0; P < kPairs; ++P)
#pragma unroll
        for (int r = 0; r < 16; ++r) mloc = fmaxf(mloc, s[P][r]);
      float mc = fmaxf(mloc * A.sl2, m);
      m = fmaxf(mc, __shfl_xor(mc, 32));
    }
    neg_m = m == -INFINITY ? FLT_MAX : -m;
  };
  // Moves the running maximum to cover page pair P's scores (rare): rescales l and the
  // accumulators by 2^(m_old - m_new).
  auto rescale = [&](const f32x16& sp, float& neg_m) {
    float mloc = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) mloc = fmaxf(mloc, sp[r]);
    float mc = fmaxf(mloc * A.sl2, m);
    mc = fmaxf(mc, __shfl_xor(mc, 32));
    const float alpha = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mc);
    l *= alpha;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) acc[cb] *= alpha;
    m = mc;
    neg_m = m == -INFINITY ? FLT_MAX : -m;
  };

  // Page pair P of step n: probabilities (consuming s[P]), step n + 1's scores of the
  // pair (from stage kread, unless last) and O^T += V^T P^T over the pair's two pages
  // from V stage vread.  V operand of page j, channel block cb: lane (channel
  // 32 cb + col, hh) reads granule 128 hh + 32 cb + col, keys in the order of the P
  // operand (element p: slot 8 (p / 4) + 4 hh + p % 4), which is the score layout.
  auto pair = [&](int P, auto kread, auto vread, int key0, f32x16 (&s)[kPairs], float& neg_m,
                  auto last_tag) {
    constexpr bool kLast = decltype(last_tag)::value;
    uint4 kpre[8];
    if constexpr (!kLast) {
#pragma unroll
      for (int c = 0; c < 8; ++c) kpre[c] = kst(kread)[2 * P + (col >> 4)][(2 * c + hh) * 16 + (col & 15)];
    }
    // Probabilities against the current maximum.  A probability above 2^kTau (the
    // maximum is stale by more than kTau, or this is a new row's first real score)
    // makes this lane's sum of the pair exceed 2^kTau: the wave then moves the maximum
    // to the pair's own and takes them again, before any product has used them.
    float p[16], ps;
    auto take = [&]() {
#pragma unroll
      for (int r = 0; r < 16; ++r) p[r] = __builtin_amdgcn_exp2f(fmaf(s[P][r], A.sl2, neg_m));
      const float t0 = (p[0] + p[1]) + (p[2] + p[3]), t1 = (p[4] + p[5]) + (p[6] + p[7]);
      const float t2 = (p[8] + p[9]) + (p[10] + p[11]), t3 = (p[12] + p[13]) + (p[14] + p[15]);
      ps = (t0 + t1) + (t2 + t3);
    };
    take();
    if (__ballot(!(ps <= kSumTau))) {
      rescale(s[P], neg_m);
      take();
    }
    l += ps;
    uint4 pa, pb;
    pa.x = pack_bf16x2(p[0], p[1]);
    pa.y = pack_bf16x2(p[2], p[3]);
    pa.z = pack_bf16x2(p[4], p[5]);
    pa.w = pack_bf16x2(p[6], p[7]);
    pb.x = pack_bf16x2(p[8], p[9]);
    pb.y = pack_bf16x2(p[10], p[11]);
    pb.z = pack_bf16x2(p[12], p[13]);
    pb.w = pack_bf16x2(p[14], p[15]);
    // Step n + 1's scores of the pair (a chain of 8 dependent MFMAs) interleaved with the
    // pair's PV products (8 independent ones), so the chain's latency is covered.
    if constexpr (!kWide) __builtin_amdgcn_s_setprio(1);
    f32x16 qs;
#pragma unroll
    for (int r = 0; r < 16; ++r) qs[r] = 0.f;
    uint32_t mk[2][4];
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int e = 0; e < 4; ++e) mk[jj][e] = ~0u;
    if constexpr (kLast) {
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const int valid = kv1 - key0 - (2 * P + jj) * kPage;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int s0 = 8 * ((2 * e) / 4) + 4 * hh + (2 * e) % 4;
          const int s1 = 8 * ((2 * e + 1) / 4) + 4 * hh + (2 * e + 1) % 4;
          mk[jj][e] = (s0 < valid ? 0x0000FFFFu : 0u) | (s1 < valid ? 0xFFFF0000u : 0u);
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      if constexpr (!kLast) {
        qs = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kpre[c]), qop[c], qs, 0, 0, 0);
      }
      const int jj = c >> 2, cb = c & 3;
      uint4 vo = vst(vread)[2 * P + jj][128 * hh + 32 * cb + col];
      if constexpr (kLast) {
        vo.x &= mk[jj][0];
        vo.y &= mk[jj][1];
        vo.z &= mk[jj][2];
        vo.w &= mk[jj][3];
      }
      acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vo), as_bf16x8(jj == 0 ? pa : pb),
                                                        acc[cb], 0, 0, 0);
    }
    if constexpr (!kLast) s[P] = qs;
  };

  // Wave priority.  Wide form: 1 from a step's opening barrier through its first page pair,
  // 0 for the second.  The two waves of a SIMD otherwise share issue by age, so the older
  // one ran each step's pairs ~40% faster than its partner and then idled at the barrier
  // while the younger finished alone; dropping the priority of a wave once it is half-way
  // through lets a lagging partner catch up within the step.  Narrow form: the two waves
  // belong to different workgroups; 1 for the products, 0 for the probabilities.
  if constexpr (kWide) __builtin_amdgcn_s_setprio(1);

  f32x16 sc[kPairs];
#pragma unroll
  for (int P = 0; P < kPairs; ++P) qk_pair(S0{}, P, sc[P]);
  if (last == 0) __syncthreads();  // the epilogue reuses the K stages; else a step's barrier is between
  // Step n copies step n + 3 into the stages that step n - 1 finished with; at its end
  // only those four copies may be in flight (vmcnt(4)): step n + 2's have landed.
  // Past the last key nothing is copied, and the wait is for all.
  auto step = [&](int n, auto r_tag, auto all_tag) {
    constexpr bool kAll = decltype(all_tag)::value;
    constexpr int r = decltype(r_tag)::value;
    using KRead = std::integral_constant<int, (r + 1) & 3>;
    using VRead = std::integral_constant<int, r>;
    using Copy = std::integral_constant<int, (r + 3) & 3>;
    const int key0 = kv0 + n * kStepKeys;
    const bool cp = kAll || n + 3 <= last;
    if (cp) {
      const uint64_t o = page_off(n + 3);
      copy_tile(k_lane, kst(Copy{}), o);
      copy_tile(v_lane, vst(Copy{}), o);
    }
    float neg_m;
    if constexpr (!kWide) __builtin_amdgcn_s_setprio(0);
    prepare(key0, sc, neg_m, n == 0);
    pair(0, KRead{}, VRead{}, key0, sc, neg_m, std::false_type{});
    if constexpr (kWide) {
      __builtin_amdgcn_s_setprio(0);
      pair(1, KRead{}, VRead{}, key0, sc, neg_m, std::false_type{});
    }
    if (cp) __builtin_amdgcn_s_waitcnt(0xF74);
    else __builtin_amdgcn_s_waitcnt(0xF70);
    __syncthreads();
    if constexpr (kWide) __builtin_amdgcn_s_setprio(1);
  };
  int n0 = 0;
  for (; n0 + 6 <= last; n0 += 4) {
    step(n0, S0{}, std::true_type{});
    step(n0 + 1, S1{}, std::true_type{});
    step(n0 + 2, S2{}, std::true_type{});
    step(n0 + 3, S3{}, std::true_type{});
  }
  for (; n0 < last; n0 += 4) {
    step(n0, S0{}, std::false_type{});
    if (n0 + 1 < last) step(n0 + 1, S1{}, std::false_type{});
    if (n0 + 2 < last) step(n0 + 2, S2{}, std::false_type{});
    if (n0 + 3 < last) step(n0 + 3, S3{}, std::false_type{});
  }
  {
    const int key0 = kv0 + last * kStepKeys;
    float neg_m;
    prepare(key0, sc, neg_m, last == 0);
    auto tail = [&](auto v_tag) {
      pair(0, S0{}, v_tag, key0, sc, neg_m, std::true_type{});
      if constexpr (kWide) pair(1, S0{}, v_tag, key0, sc, neg_m, std::true_type{});
    };
    switch (last & 3) {
      case 0: tail(S0{}); break;
      case 1: tail(S1{}); break;
      case 2: tail(S2{}); break;
      default: tail(S3{}); break;
    }
  }

  // Epilogue.  Row col's sum over both lane halves; a lane holds, per channel block, 16
  // channels of its row (runs of 4 at 32 cb + 8 e + 4 hh).  The rows go through LDS so that
  // each store instruction writes whole rows (16 lanes x 16 B of each of four): K stages
  // are free (the last step reads V only, and no copy is in flight), 8 KiB per wave, rows
  // of 256 B whose 16-byte granules are XORed with the row against bank conflicts.
  const float ls = l + __shfl_xor(l, 32);
  const float inv = ls > 0.f ? 1.f / ls : 0.f;
  uint4* const buf = (kWide ? (wave < 4 ? (wave < 2 ? &ldk0[0][0] : &ldk1[0][0])
                                        : (wave < 6 ? &ldk2[0][0] : &ldk3[0][0])) + (wave & 1) * 512
                            : (wave < 2 ? (wave < 1 ? &ldk0[0][0] : &ldk1[0][0])
                                        : (wave < 3 ? &ldk2[0][0] : &ldk3[0][0])));
  const int sw = col & 15;
  auto wave_sync = [&]() {  // LDS operations of one wave complete in order
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  if (nsplit > 1) {
    // One split of the rows: normalised float32 partials, 64 channels at a time, and the
    // base-2 log-sum-exp; chunk_merge_kernel combines the splits after this launch.
    const size_t prow = size_t(part) * kRows + 32 * wave;
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
      wave_sync();
#pragma unroll
      for (int cb = 2 * h2; cb < 2 * h2 + 2; ++cb)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          *reinterpret_cast<f32x4*>(&buf[col * 16 + ((8 * (cb & 1) + 2 * e + hh) ^ sw)]) =
              f32x4{acc[cb][4 * e] * inv, acc[cb][4 * e + 1] * inv, acc[cb][4 * e + 2] * inv,
                    acc[cb][4 * e + 3] * inv};
      wave_sync();
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int r = 4 * i + (lane >> 4), c = lane & 15;
        *reinterpret_cast<uint4*>(A.part_o + (prow + r) * kDim + 64 * h2 + 4 * c) =
            buf[r * 16 + (c ^ (r & 15))];
      }
    }
    // -inf only where the row saw no key: a NaN sum gives a NaN, which the merge keeps.
    if (hh == 0) A.part_lse[prow + col] = ls == 0.f ? -INFINITY : m + log2f(ls);
    return;
  }
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint2 w;
      w.x = pack_bf16x2(acc[cb][4 * e] * inv, acc[cb][4 * e + 1] * inv);
      w.y = pack_bf16x2(acc[cb][4 * e + 2] * inv, acc[cb][4 * e + 3] * inv);
      reinterpret_cast<uint2*>(&buf[col * 16 + ((4 * cb + e) ^ sw)])[hh] = w;
    }
  wave_sync();
  const size_t head0 = size_t(g) * G;
  const uint32_t inv_g = (65536u + G - 1) / G;  // r / G = r * inv_g >> 16 for r < 256
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int rl = 4 * i + (lane >> 4), c = lane & 15;
    const uint32_t r = r_first + 32 * wave + rl;
    const int tk = q0 + int(r * inv_g >> 16);
    if (tk < q1) {
      const size_t orow = size_t(row0 + tk) * A.hq + head0 + (r - (r * inv_g >> 16) * G);
      *reinterpret_cast<uint4*>(A.out + orow * kDim + 8 * c) = buf[rl * 16 + (c ^ (rl & 15))];
    }
  }
  if (A.lse && hh == 0 && ok)
    A.lse[size_t(row0 + t_tok) * A.hq + head0 + head] = ls > 0.f ? (m + log2f(ls)) * kLn2 : -INFINITY;
}

}  // namespace

hipError_t launch_chunk(const KvLayout& L, const Plan& P, void* ws, const void* q,
                        const int32_t* bt, int32_t stride, float scale, void* out, float* lse,
                        hipStream_t s) {
  if (P.info.n_chunk == 0) return hipSuccess;
  char* w = static_cast<char*>(ws);
  ChunkArgs A;
  A.k_cache = static_cast<const uint16_t*>(L.desc.k_cache);
  A.v_cache = static_cast<const uint16_t*>(L.desc.v_cache);
  A.units = reinterpret_cast<const int32_t*>(w + P.off_units) + size_t(P.info.n_single) * kUnitInts;
  A.tiles = reinterpret_cast<const int32_t*>(w + P.off_tiles);
  A.form = P.chunk_form;
  A.half_tokens = (kTileRows - 1) / P.group + 1;
  for (int x = 0; x < kNumXcds; ++x) {
    A.xcd_first[x] = P.xcd_map[size_t(2 * x)];
    A.xcd_count[x] = P.xcd_map[size_t(2 * x + 1)] * (P.chunk_form == kBothHalves ? 2 : 1);
  }
  A.bt = bt;
  A.q = static_cast<const uint16_t*>(q);
  A.out = static_cast<uint16_t*>(out);
  A.lse = lse;
  A.part_o = reinterpret_cast<float*>(w + P.off_chunk_o);
  A.part_lse = reinterpret_cast<float*>(w + P.off_chunk_lse);
  A.bt_stride = stride;
  A.hkv = P.num_kv_heads;
  A.hq = P.num_q_heads;
  A.group = P.group;
  A.sl2 = scale * kLog2e;
  if (P.chunk_form != kUnits)
    hipLaunchKernelGGL(chunk_kernel<kNarrowWaves>, dim3(unsigned(P.chunk_grid)),
                       dim3(64 * kNarrowWaves), 0, s, A);
  else
    hipLaunchKernelGGL(chunk_kernel<kWideWaves>, dim3(unsigned(P.chunk_grid)),
                       dim3(64 * kWideWaves), 0, s, A);
  return hipGetLastError();
}

}  // namespace libra
