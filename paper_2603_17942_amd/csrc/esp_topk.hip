// Fused vocabulary softmax + Top-K' of the mask-row logits (paper Sec. 2 Eq. 2, Sec. 3.3).
//
// Each logit row is read exactly once, by independent wavefronts and without a barrier.
// Pass 1 (k_topk_stream): a wave streams one segment of one row in blocks of 2048 logits
// (32 per lane, float4 loads, the next block in flight while the current one is reduced).
//   * softmax statistics stay lane-local (running maximum and rescaled sum of exponentials) and
//     are combined across the wave once, at the end of the segment;
//   * the K' best (value desc, id asc) live in a list spread over the lanes (lane j holds the
//     j-th best).  A block is only looked at when its maximum reaches the current K'-th value,
//     which after the first block is rare (about K' ln(n/K') times per n logits), so the common
//     path per logit is one max, one fma, one exp and one add.  The first block is filtered by a bound
//     that at least K' of its 64 lane maxima reach, and at most two more unless maxima are equal; up to 64
//     logits that reach it are ranked at once, more (ties) are inserted one by one like those of later blocks.
// Pass 2 (k_topk_merge): one wave per row merges the segment statistics (online-softmax rule) and
// the segments' sorted lists (at most 64 segments, one per lane: K' rounds of a wave-wide best-head
// search); p = min(1, exp(v - max) / sum) in fp32.
#include <algorithm>
#include <climits>
#include <mutex>

#include "esp_internal.h"

namespace {

constexpr int BLOCK = 2048;            // logits per wave and iteration
constexpr int PER_LANE = BLOCK / 64;
constexpr float LOG2E_F = 1.4426950408889634f;

__device__ __forceinline__ bool better(float av, int ai, float bv, int bi) {
  return av > bv || (av == bv && ai < bi);
}
__device__ __forceinline__ float readlane_f(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// The K' best so far, lane j < kp holding the j-th; lanes >= kp hold (-inf, INT_MAX).
struct LaneList {
  float v;
  int id;
  float last_v;   // entry kp-1 (wave-uniform)
  int last_id;
};
__device__ __forceinline__ void list_init(LaneList& L) {
  L.v = -INFINITY; L.id = 0x7fffffff; L.last_v = -INFINITY; L.last_id = 0x7fffffff;
}
// insert (v, id), known to be better than the last entry; v, id wave-uniform
__device__ __forceinline__ void list_insert(LaneList& L, float v, int id, int kp, int lane) {
  const bool mine_better = lane < kp && better(L.v, L.id, v, id);
  const int pos = __popcll(__builtin_amdgcn_ballot_w64(mine_better));   // the better entries form a prefix
  const float up_v = __shfl_up(L.v, 1, 64);
  const int up_i = __shfl_up(L.id, 1, 64);
  if (lane < kp) {
    if (lane == pos) { L.v = v; L.id = id; }
    else if (lane > pos) { L.v = up_v; L.id = up_i; }
  }
  L.last_v = readlane_f(L.v, kp - 1);
  L.last_id = __builtin_amdgcn_readlane(L.id, kp - 1);
}

__device__ __forceinline__ int lanes_below(unsigned long long ballot) {   // set bits below this lane
  return __builtin_amdgcn_mbcnt_hi((unsigned)(ballot >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)ballot, 0u));
}

// reductions over the wave, returned to all lanes: data-parallel-primitive moves, which lanes without a
// source (`idle` = the operation's neutral value) pass through, instead of LDS exchanges
template <typename Op>
__device__ __forceinline__ float wave_reduce_dpp(float x, float idle, Op op) {
  const int id = __float_as_int(idle);
#define ESP_DPP_STEP(ctrl) x = op(x, __int_as_float(__builtin_amdgcn_update_dpp(id, __float_as_int(x), ctrl, 0xf, 0xf, false)))
  ESP_DPP_STEP(0x111);   // row_shr:1, 2, 4, 8
  ESP_DPP_STEP(0x112);
  ESP_DPP_STEP(0x114);
  ESP_DPP_STEP(0x118);
#undef ESP_DPP_STEP
  // lane 15 of each row of 16 holds the row's result
  return op(op(readlane_f(x, 15), readlane_f(x, 31)), op(readlane_f(x, 47), readlane_f(x, 63)));
}
__device__ __forceinline__ float wave_max_dpp(float x) {
  return wave_reduce_dpp(x, -INFINITY, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float wave_sum_dpp(float x) {
  return wave_reduce_dpp(x, 0.f, [](float a, float b) { return a + b; });
}

// A bound that at least kp of the 64 lane values reach and, unless values are equal, at most two more; -inf when
// fewer than kp are finite.  lanes = how many reach it, top = the wave's maximum.  The distance below the top is
// found to a factor of eight first and then by bisection: over the values' whole range a single lane of large
// finite masks (-1e9) uses up all halvings, every logit of the block reaches the bound and is inserted one by
// one (64 rows of 128256: 41 us against 13).
__device__ __forceinline__ float low_bound(float x, float top, int kp, int& lanes) {
  lanes = 0;
  if (__popcll(__builtin_amdgcn_ballot_w64(x > -INFINITY)) < kp) return -INFINITY;
  float width = 8.f, lo = top - width, hi = top;
#pragma unroll 1
  while ((lanes = __popcll(__builtin_amdgcn_ballot_w64(x >= lo))) < kp) {
    if (!(width < 1e37f)) return -INFINITY;              // infinities, or the whole range of the type
    hi = lo;
    width *= 8.f;
    lo = top - width;
  }
#pragma unroll 1
  for (int it = 0; it < 16 && lanes > kp + 2; ++it) {
    const float mid = 0.5f * (lo + hi);
    const int reach = __popcll(__builtin_amdgcn_ballot_w64(x >= mid));
    if (reach >= kp) { lo = mid; lanes = reach; } else hi = mid;
  }
  return lo;
}

// the next larger value; NaN, which nothing reaches, after infinity
__device__ __forceinline__ float next_above(float x) {
  const int bits = __float_as_int(x);
  return bits == INT_MIN ? __int_as_float(1) : __int_as_float(bits >= 0 ? bits + 1 : bits - 1);
}

// Offer the values of one register slot (one per lane) to the list: every lane whose value
// reaches the bound is examined in turn (wave-uniform loop over the ballot).
__device__ __forceinline__ void offer(LaneList& L, float v, int my_id, float& bound, float floor_bound, int kp,
                                      int lane) {
  unsigned long long mask = __builtin_amdgcn_ballot_w64(v >= bound);
  while (mask) {
    const int l = __builtin_ctzll(mask);
    mask &= mask - 1;
    const float cv = readlane_f(v, l);
    const int cid = __builtin_amdgcn_readlane(my_id, l);
    if (better(cv, cid, L.last_v, L.last_id)) {
      list_insert(L, cv, cid, kp, lane);
      bound = fmaxf(floor_bound, L.last_v);
      mask &= __builtin_amdgcn_ballot_w64(v >= bound);
    }
  }
}

// record per (row, segment): [max, sum, v_0..v_{kp-1}, id_0..id_{kp-1}] as 2 + 2*kp words
__global__ __launch_bounds__(256) void k_topk_stream(const float* __restrict__ logits, int rows, int vocab, int kp,
                                                     int nseg, int seg_len, float* __restrict__ seg_rec,
                                                     const int32_t* __restrict__ row_map) {
  __shared__ float cand_v[4][64];
  __shared__ int cand_id[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int item = blockIdx.x * 4 + wave;
  if (item >= rows * nseg) return;                      // (waves work alone: no barrier below)
  const int row = item / nseg, seg = item % nseg;
  const int start = seg * seg_len, end = min(vocab, start + seg_len);
  const float* p = logits + (size_t)(row_map ? max(row_map[row], 0) : row) * vocab;
  const bool vec4 = (vocab & 3) == 0 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0;
  const int nblocks = (max(end - start, 0) + BLOCK - 1) / BLOCK;

  // element e of float4 i of the lane sits at block_base + i*256 + lane*4 + e
  float nxt[PER_LANE], cur[PER_LANE];
  auto load_block = [&](int b, float (&dst)[PER_LANE]) {
    const int base = start + b * BLOCK + lane * 4;
    if (vec4 && start + (b + 1) * BLOCK <= end) {
#pragma unroll
      for (int i = 0; i < PER_LANE / 4; ++i) {
        const f32x4_t q = *reinterpret_cast<const f32x4_t*>(p + base + i * 256);
        dst[4 * i] = q[0]; dst[4 * i + 1] = q[1]; dst[4 * i + 2] = q[2]; dst[4 * i + 3] = q[3];
      }
    } else {
#pragma unroll
      for (int i = 0; i < PER_LANE; ++i) {
        const int idx = base + (i >> 2) * 256 + (i & 3);
        dst[i] = idx < end ? p[idx] : -INFINITY;
      }
    }
  };

  LaneList L;
  list_init(L);
  float m = -INFINITY, s = 0.f;       // lane-local running maximum and sum of 2^((v - m) log2 e)
  // gate: what a block's maximum has to reach to be looked at.  A later block's ids are higher than all listed ones,
  // so there it has to exceed the bound (rows of one repeated value: 4.2 ms for 1024 rows of 128256 without that)
  float floor_bound = -INFINITY, bound = -INFINITY, gate = -INFINITY;
  if (nblocks > 0) load_block(0, nxt);
  for (int b = 0; b < nblocks; ++b) {
#pragma unroll
    for (int i = 0; i < PER_LANE; ++i) cur[i] = nxt[i];
    if (b + 1 < nblocks) load_block(b + 1, nxt);
    float bmax = cur[0];
#pragma unroll
    for (int i = 1; i < PER_LANE; ++i) bmax = fmaxf(bmax, cur[i]);
    const float m_new = fmaxf(m, bmax);
    if (m_new > -INFINITY) {
      // Over a large finite mask (1e30, the type's lowest value) the rounded product is off by more than the
      // exponents exp2 can take: a lane that holds nothing else adds 0, not infinity.
      const float mb = fmaxf(m_new * LOG2E_F, -0x1p31f);
      float acc = s * __builtin_amdgcn_exp2f(m * LOG2E_F - mb);   // m = -inf: 0
#pragma unroll
      for (int i = 0; i < PER_LANE; ++i) acc += __builtin_amdgcn_exp2f(fmaf(cur[i], LOG2E_F, -mb));
      s = acc;
      m = m_new;
    }
    if (b == 0) {
      int lanes;
      floor_bound = low_bound(bmax, wave_max_dpp(bmax), kp, lanes);
      bound = gate = floor_bound;
      // the values that reach the bound (kp or a few more) are collected in LDS and ranked together
      // (not where most lanes are tied at it: equal values by the thousand are offered below)
      int n = 0;
      if (floor_bound > -INFINITY && lanes <= 48) {
#pragma unroll
        for (int i = 0; i < PER_LANE; ++i) {
          const bool in = cur[i] >= floor_bound;
          const unsigned long long mask = __builtin_amdgcn_ballot_w64(in);
          if (mask == 0ull) continue;                    // most registers hold none
          const int at = n + lanes_below(mask);
          if (in && at < 64) { cand_v[wave][at] = cur[i]; cand_id[wave][at] = start + lane * 4 + (i >> 2) * 256 + (i & 3); }
          n += __popcll(mask);
        }
      }
      if (n > 0 && n <= 64) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const float v = lane < n ? cand_v[wave][lane] : -INFINITY;
        const int id = lane < n ? cand_id[wave][lane] : 0x7fffffff;
        int rank = 0;
        for (int l = 0; l < n; ++l) rank += better(readlane_f(v, l), __builtin_amdgcn_readlane(id, l), v, id) ? 1 : 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (lane < n) { cand_v[wave][rank] = v; cand_id[wave][rank] = id; }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (lane < kp) { L.v = cand_v[wave][lane]; L.id = cand_id[wave][lane]; }   // n >= kp
        L.last_v = readlane_f(L.v, kp - 1);
        L.last_id = __builtin_amdgcn_readlane(L.id, kp - 1);
        bound = fmaxf(floor_bound, L.last_v);
        gate = next_above(bound);
        continue;
      }
    }
    if (__builtin_amdgcn_ballot_w64(bmax >= gate) != 0ull) {
      const int base = start + b * BLOCK + lane * 4;
#pragma unroll
      for (int i = 0; i < PER_LANE; ++i) offer(L, cur[i], base + (i >> 2) * 256 + (i & 3), bound, floor_bound, kp, lane);
      gate = next_above(bound);
    }
  }
  // wave-wide statistics in the natural-exponent convention: sum of exp(v - max)
  const float wm = wave_max_dpp(m);
  const float contrib = m > -INFINITY ? s * __builtin_amdgcn_exp2f((m - wm) * LOG2E_F) : 0.f;
  const float ws = wave_sum_dpp(contrib);
  float* out = seg_rec + ((size_t)row * nseg + seg) * (2 + 2 * kp);
  if (lane == 0) { out[0] = wm; out[1] = ws; }
  if (lane < kp) {
    out[2 + lane] = L.v;
    reinterpret_cast<int*>(out)[2 + kp + lane] = L.id;
  }
}

// one wave per row: the segments' lists are sorted, so lane c walks segment c's list and the wave
// takes the best head (value desc, id asc) K' times -- a 64-way merge of sorted lists.  The lists are
// brought into LDS once: read where they are, every round would expose a memory latency.
__global__ __launch_bounds__(64) void k_topk_merge(const float* __restrict__ seg_rec, int kp, int nseg,
                                                   int32_t* __restrict__ ids, float* __restrict__ probs) {
  extern __shared__ float lists[];                                      // [2 kp][64]
  const int lane = threadIdx.x, row = blockIdx.x;
  const int stride = 2 + 2 * kp;
  const bool have = lane < nseg;                                        // this lane's segment (nseg <= 64)
  const float* e = seg_rec + ((size_t)row * nseg + min(lane, nseg - 1)) * stride;
  const float smax = have ? e[0] : -INFINITY, ssum = have ? e[1] : 0.f;
#pragma unroll 4
  for (int j = 0; j < 2 * kp; ++j) lists[j * 64 + lane] = e[2 + j];
  const float gmax = wave_max_dpp(smax);
  const float tot = wave_sum_dpp(smax > -INFINITY ? ssum * expf(smax - gmax) : 0.f);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  int pos = 0;                                                          // next unread entry of the list
  float hv = have ? lists[lane] : -INFINITY;
  int hi = __float_as_int(lists[kp * 64 + lane]);
  float out_v = -INFINITY;
  int out_i = -1;
  for (int j = 0; j < kp; ++j) {
    const float best = wave_max_dpp(hv);
    if (best == -INFINITY) break;                                       // empty slots never win
    unsigned long long top = __builtin_amdgcn_ballot_w64(hv == best);
    int win = __builtin_ctzll(top);
    int bi = __builtin_amdgcn_readlane(hi, win);
    for (top &= top - 1; top; top &= top - 1) {                         // equal values: the lowest id
      const int l = __builtin_ctzll(top), oi = __builtin_amdgcn_readlane(hi, l);
      if (oi < bi) { bi = oi; win = l; }
    }
    if (lane == j) { out_v = best; out_i = bi; }
    if (lane == win) {
      ++pos;
      hv = pos < kp ? lists[pos * 64 + lane] : -INFINITY;
      hi = pos < kp ? __float_as_int(lists[(kp + pos) * 64 + lane]) : -1;
    }
  }
  if (lane < kp) {
    ids[(size_t)row * kp + lane] = out_i;
    // the sum's own term at the maximum, exp2(fma(m, log2 e, -round(m log2 e))), can lie a few units in the last place
    // below 1: a row with nearly all probability on one token would hand out more than 1.  NaN stays NaN.
    const float p = expf(out_v - gmax) / tot;
    probs[(size_t)row * kp + lane] = out_i < 0 ? 0.f : (p > 1.f ? 1.f : p);
  }
}

// Segments per row, at most 64 (the merge gives each a lane).  Where that makes up to 4096 waves (four per SIMD,
// all resident at once), a row of up to 64 blocks (131072 logits) gets a wave per block: every load of the launch is
// then in flight from the start (64 rows of 128256: 14.8 us against 16.8 us with two blocks a wave).  Longer rows
// get two blocks a wave at any row count (151936: 38 segments; 64 rows 18.3 us).  With more waves than that the
// fixed cost per wave counts and about 2048 waves walk several blocks each (256 rows: 33.4 us against 36.3 us with
// 4096 waves).  Between, only 64 and 256 rows were compared: at 128256 the rule turns at 66 rows, and 65 rows take
// 12.8 us where 80 take 19.4 us.
int topk_segments(int rows, int vocab, int* seg_len) {
  const int max_seg = std::min(64, (vocab + BLOCK - 1) / BLOCK);   // the merge gives each segment a lane
  const int waves = (int64_t)rows * max_seg <= 4096 ? 4096 : 2048;
  int nseg = std::max(1, std::min(max_seg, (waves + rows - 1) / rows));
  int len = ((vocab + nseg - 1) / nseg + BLOCK - 1) / BLOCK * BLOCK;
  nseg = (vocab + len - 1) / len;
  *seg_len = len;
  return nseg;
}

// ---- entry point for callers that cannot allocate ---------------------------------------------
// Per-(row, segment) statistics and candidate lists of the two-pass Top-K' in a file-scope device
// array instead of a caller workspace.  Every GPU the library runs on holds its own copy of the
// array (at its own address) until the process ends; the host-side name is only a handle for
// hipGetSymbolAddress, whose result (per device) is what the kernels receive.
constexpr int STATIC_MAX_ROWS = 128;
constexpr size_t STATIC_SCRATCH_FLOATS = (size_t)STATIC_MAX_ROWS * 64 * (2 + 2 * ESP_MAX_TOPK);   // 2.06 MiB
static __device__ __align__(256) __attribute__((used)) float scratch[STATIC_SCRATCH_FLOATS];

constexpr int MAX_DEVICES = 64;
static std::mutex g_scratch_mutex;
static float* g_scratch_ptr[MAX_DEVICES] = {};   // device address of `scratch` on each device, 0 = not looked up yet

// device address of the array on the current device (looked up once per device)
static hipError_t static_scratch(float** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = static_cast<float*>(p);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace

extern "C" esp_status esp_softmax_topk_static(void* stream, const float* logits, int32_t rows, int32_t vocab,
                                              int32_t Kp, int32_t* ids, float* probs) {
  if (!logits || !ids || !probs) return ESP_EINVAL;
  if (rows < 1 || vocab < 1 || Kp < 1 || Kp > ESP_MAX_TOPK || Kp > vocab) return ESP_EINVAL;
  if (softmax_topk_scratch_floats(rows, vocab, Kp) > STATIC_SCRATCH_FLOATS) return ESP_ECAPACITY;
  float* ws = nullptr;
  if (static_scratch(&ws) != hipSuccess) return ESP_EDEVICE;
  // every (row, segment) record the merge pass reads is written by the stream pass of the same
  // call, so nothing of an earlier call's contents has to be cleared
  if (launch_softmax_topk((hipStream_t)stream, logits, rows, vocab, Kp, ids, probs, ws, nullptr) != hipSuccess)
    return ESP_EDEVICE;
  return ESP_OK;
}

size_t softmax_topk_scratch_floats(int rows, int vocab, int kp) {
  int max_seg = std::min(64, (vocab + BLOCK - 1) / BLOCK);   // upper bound of the segment count for any row count
  return (size_t)rows * max_seg * (2 + 2 * kp);
}

hipError_t launch_softmax_topk(hipStream_t st, const float* logits, int rows, int vocab, int kp, int32_t* ids,
                               float* probs, float* ws, const int32_t* row_map) {
  if (rows <= 0) return hipSuccess;
  int seg_len = 0;
  const int nseg = topk_segments(rows, vocab, &seg_len);
  const int items = rows * nseg;
  hipLaunchKernelGGL(k_topk_stream, dim3((items + 3) / 4), dim3(256), 0, st, logits, rows, vocab, kp, nseg, seg_len,
                     ws, row_map);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_topk_merge, dim3(rows), dim3(64), (size_t)2 * kp * 64 * 4, st, ws, kp, nseg, ids, probs);
  return hipGetLastError();
}
