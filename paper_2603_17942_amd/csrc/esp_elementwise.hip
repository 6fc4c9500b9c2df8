// Glue kernels of the ESP decode step: block assembly, norms, rotary + KV append,
// argmax, KV copies, mask-vector init / update.  All HBM-light; one pass over [rows, width].
#include <algorithm>

#include "esp_internal.h"

#define ESP_DISPATCH(dtype, ...)          \
  do {                                    \
    if ((dtype) == ESP_F32) {             \
      using T = float;                    \
      __VA_ARGS__;                        \
    } else {                              \
      using T = bf16_t;                   \
      __VA_ARGS__;                        \
    }                                     \
  } while (0)

// no short circuit: the loads are issued together
__device__ __forceinline__ bool seq_valid(const KvDev& kv, int L, int base, int cap, int n_rows) {
  return (L >= 0) & (L <= kv.len_bound) & (n_rows >= 0) & (L + n_rows <= cap) & (base >= 0) & ((base & 63) == 0) &
         ((int64_t)(uint32_t)base + (uint32_t)cap <= kv.capacity);   // a negative one has failed already
}
__device__ __forceinline__ bool seq_ok(const KvDev& kv, int seq, int n_rows) {
  return seq_valid(kv, kv.len[seq], kv.base[seq], kv.seq_cap[seq], n_rows);
}

// 1 / rms of a row of width d, from the threads' sums of squares
__device__ __forceinline__ float rms_scale(float ss, int d, float eps, float* red) {
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
  for (int w = 0; w < (int)blockDim.x >> 6; ++w) tot += red[w];
  return 1.0f / sqrtf(tot / (float)d + eps);
}

__device__ __forceinline__ float block_sum_256(float v, float* red) {
  v = wave_sum(v);
  int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float t = red[0] + red[1] + red[2] + red[3];
  __syncthreads();
  return t;
}

// ---- block assembly (Sec. 3.1, Sec. 3.3): h0 rows and the per-row rotary table ---------------
// Packed rows of a batch (BlockDev): one workgroup per sequence adds up the row counts of the sequences before it
// and writes its own rows' places.  A sequence that is not valid (or a count that does not fit) has no rows; its tree
// rows follow the block alone, as in node_row.
__global__ __launch_bounds__(256) void k_live_rows(BlockDev b, KvDev kv, int max_nodes, GateUpRule gate_up) {
  __shared__ float red[4];
  const int seq = blockIdx.x;
  auto rows_of = [&](int s) {
    const int nr = b.n_rows[s];
    return nr <= b.rows_per_seq && seq_ok(kv, s, nr) ? nr : 0;
  };
  auto nodes_of = [&](int s) {
    const int nn = b.n_nodes[s];
    return nn >= 0 && nn <= b.n_rows[s] && b.n_rows[s] <= b.rows_per_seq ? min(nn, max_nodes) : 0;
  };
  float r0 = 0.f, q0 = 0.f;             // counts below 2^24: exact
  for (int s = threadIdx.x; s < seq; s += 256) {
    r0 += (float)rows_of(s);
    q0 += (float)nodes_of(s);
  }
  const int first = (int)block_sum_256(r0, red), node0 = (int)block_sum_256(q0, red);
  const int nr = rows_of(seq);
  for (int r = threadIdx.x; r < b.rows_per_seq; r += 256) {
    const int row = seq * b.rows_per_seq + r;
    b.packed_row()[row] = r < nr ? first + r : -1;
    if (r < nr) b.live_rows()[first + r] = row;
  }
  if (threadIdx.x == 0) {
    b.seq_row0()[seq] = first;
    b.seq_node0()[seq] = node0;
    if (seq + 1 == b.batch) {
      b.n_live()[0] = first + nr;
      b.n_live()[1] = node0 + nodes_of(seq);
      const int tile = gate_up.cheapest_launched(first + nr);
      for (int t = 0; t < GU_TILES; ++t) b.n_live()[2 + t] = t == tile ? first + nr : 0;
    }
  }
}

hipError_t launch_live_rows(hipStream_t st, const BlockDev& b, const KvDev& kv, int max_nodes, const GateUpRule& gate_up) {
  hipLaunchKernelGGL(k_live_rows, dim3(b.batch), dim3(256), 0, st, b, kv, max_nodes, gate_up);
  return hipGetLastError();
}

template <typename T> struct Pack4;
template <> struct Pack4<float> {
  using Raw = f32x4_t;
  static __device__ __forceinline__ f32x4_t value(Raw v) { return v; }
  static __device__ __forceinline__ void store(float* p, f32x4_t v) { *reinterpret_cast<f32x4_t*>(p) = v; }
  static __device__ __forceinline__ f32x4_t load(const float* p) { return *reinterpret_cast<const f32x4_t*>(p); }
};
template <> struct Pack4<bf16_t> {
  using Raw = bf16x4_t;
  static __device__ __forceinline__ f32x4_t value(Raw i) {
    f32x4_t o = {(float)i[0], (float)i[1], (float)i[2], (float)i[3]};
    return o;
  }
  static __device__ __forceinline__ void store(bf16_t* p, f32x4_t v) {
    bf16x4_t o = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
    *reinterpret_cast<bf16x4_t*>(p) = o;
  }
  static __device__ __forceinline__ f32x4_t load(const bf16_t* p) { return value(*reinterpret_cast<const bf16x4_t*>(p)); }
};

// Gather lists for the LM head over node rows: logical row m = seq*max_nodes + i; in a batch with packed rows the
// tree rows that are there come first, one after the other, and the rest of the lists is marked unused.
__device__ __forceinline__ void node_row(const BlockDev& b, const KvDev& kv, const NodeLists& n, int m) {
  if (m >= b.batch * n.max_nodes) return;
  const int seq = m / n.max_nodes, i = m % n.max_nodes;
  const int nn = b.n_nodes[seq];
  const bool live = i < nn && nn <= b.n_rows[seq] && b.n_rows[seq] <= b.rows_per_seq;
  const int row = seq * b.rows_per_seq + (live ? i : 0);
  if (b.packed) {
    if (m >= b.n_live()[1]) { n.a_rows[m] = 0; n.out_rows[m] = -1; n.positions[m] = 0; }
    if (!live) return;
    m = b.seq_node0()[seq] + i;
  }
  n.a_rows[m] = row;
  n.out_rows[m] = live ? row : -1;
  n.positions[m] = kv.len[seq] + b.depth[row] + 1;
}

// One workgroup per block row: its embedding, its rotary table and the first layer's norm of it (threads and order of the sum as in
// k_residual_norm); the workgroups behind the rows write the LM head's gather lists.  A launch each for the norm, the lists and the
// positions of a draw cost 4.6 us a step; embedding and norm of 68 rows of 4096 12.3 + 4.7 -> 6.3 us, of 2112 27.9 + 12.6 -> 40.6.
// The table's double-precision functions take the last waves about as long as the others wait for the embedding.
// PACKED: the row behind the live ones in the projections' inputs is set to zero; no kernel of the layers writes it, and the row
// tiles load it for every row that is not there.  (A copy of the last live row keeps the matrix cores as busy as a real one, zeros
// do not, and the card is at its power limit in the large tiles: eight layers of the 8B shape on 2048 keys, 172 rows of 318 there
// 1930 -> 1672 us, 273 of 448 2142 -> 1902.  A zero row for each instead cost the loads of it: 64 of 224 rows 1392 -> 1448.)
template <typename T, bool PACKED>
__global__ __launch_bounds__(1024) void k_embed(BlockDev b, KvDev kv, const T* __restrict__ embed, const T* __restrict__ mask_embed,
                                                float* __restrict__ h, int d, int vocab, float* __restrict__ rope_tab, int hd,
                                                float theta, int32_t* status, size_t mask_seq_stride, PackedEnd end, NodeLists lists,
                                                const T* __restrict__ gain, float eps, T* __restrict__ xn) {
  __shared__ float red[16];
  const int row = blockIdx.x, tid = threadIdx.x, step = blockDim.x, behind = row - b.batch * b.rows_per_seq;
  if (behind >= 0) {
    node_row(b, kv, lists, behind * step + tid);
    return;
  }
  if (PACKED) {
    if (row == b.n_live()[0]) {
      const u32x4_t zero = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        u32x4_t* dst = reinterpret_cast<u32x4_t*>(end.rows[t] + (size_t)row * end.width[t]);
        for (int i = tid; i < end.width[t] / 8; i += step) dst[i] = zero;
      }
    }
  }
  const int seq = row / b.rows_per_seq, r = row % b.rows_per_seq;
  const int nr = b.n_rows[seq], len = kv.len[seq], j = b.mask_j[row], t = b.tok[row], depth = b.depth[row];
  const bool ok = seq_valid(kv, len, kv.base[seq], kv.seq_cap[seq], nr) && nr <= b.rows_per_seq;
  if (r == 0 && tid == 0 && !ok) atomicOr(status, ESP_DEV_LEN_OVER_BOUND);
  const bool live = ok && r < nr;
  if (lists.row_positions && tid == 0) lists.row_positions[row] = len + depth + 1;
  if (PACKED && !live) return;
  const size_t at = PACKED ? (size_t)b.packed_row()[row] : (size_t)row;
  const T* src = nullptr;
  if (live) {
    if (j > 0) {
      if (j <= b.k_masks) src = mask_embed + seq * mask_seq_stride + (size_t)(j - 1) * d;
    } else if (t < 0 || t >= vocab) {
      if (tid == 0) atomicOr(status, ESP_DEV_BAD_TOKEN);
    } else {
      src = embed + (size_t)t * d;
    }
  }
  const int d4 = d >> 2;
  auto column = [&](int i) {                             // scalar loads: the caller's rows need no more than their type's alignment
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};
    if (src)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = to_f32(src[4 * i + e]);
    return v;
  };
  f32x4_t keep = {0.f, 0.f, 0.f, 0.f};                   // this thread's first column
  if (tid < d4) keep = column(tid);
  const int half = hd >> 1;
  for (int i = step - 1 - tid; i < half; i += step) {
    // angle in double: positions reach 1e4..1e5 where an fp32 product loses the fraction
    double pos = live ? (double)(len + depth) : 0.0;
    double ang = pos * pow((double)theta, -2.0 * (double)i / (double)hd);
    rope_tab[(at * half + i) * 2 + 0] = (float)cos(ang);
    rope_tab[(at * half + i) * 2 + 1] = (float)sin(ang);
  }
  float* hr = h + at * d;
  float ss = 0.f;
  for (int i = tid; i < d4; i += step) {
    const f32x4_t v = i == tid ? keep : column(i);
    *reinterpret_cast<f32x4_t*>(hr + 4 * i) = v;
    ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
  }
  const float inv = rms_scale(ss, d, eps, red);
  for (int i = tid; i < d4; i += step) {
    const f32x4_t v = i == tid ? keep : *reinterpret_cast<const f32x4_t*>(hr + 4 * i);   // written by this thread above
    Pack4<T>::store(xn + at * d + 4 * i, v * inv * Pack4<T>::load(gain + 4 * i));
  }
}

// threads of a workgroup for a row's norm
static int norm_threads(int d) { return std::min(1024, ((d >> 2) + 63) & ~63); }

hipError_t launch_embed(hipStream_t st, int dtype, const BlockDev& b, const KvDev& kv, const void* embed,
                        const void* mask_embed, float* h, int d, int vocab, float* rope_tab, int hd,
                        float theta, int32_t* status, size_t mask_seq_stride, const PackedEnd& end, const NodeLists& lists,
                        const void* gain, float eps, void* xn) {
  const int threads = norm_threads(d), M = b.batch * b.rows_per_seq, behind = (b.batch * lists.max_nodes + threads - 1) / threads;
  ESP_DISPATCH(dtype, hipLaunchKernelGGL((b.packed ? k_embed<T, true> : k_embed<T, false>), dim3(M + behind), dim3(threads), 0, st, b, kv,
                                         (const T*)embed, (const T*)mask_embed, h, d, vocab, rope_tab, hd, theta, status,
                                         mask_seq_stride, end, lists, (const T*)gain, eps, (T*)xn));
  return hipGetLastError();
}

// ---- residual add of split-K partials + RMSNorm ------------------------------------------------
// One workgroup per row; a thread owns float4 columns (one each up to d = 4096).  The kernel is bound by the
// fp32 partials it reads (S * d * 4 bytes per row), so the split count is a template parameter: all S loads of
// a column are in flight before the first is waited for, and the row stays in registers between the two
// passes.  d must be a multiple of 4.  d = 4096: 4.4 us at one row, 5.7 us at 68 rows (8 partials, 9 MB), 11 to
// 13 us at 320 (42 MB); with a running split count and the row read back: 12 to 13 us at 320.
// v + the S partials at p, p + stride, ..., added in split order
template <int S>
__device__ __forceinline__ f32x4_t add_splits(f32x4_t v, const float* __restrict__ p, size_t stride) {
  f32x4_t x[S];
#pragma unroll
  for (int s = 0; s < S; ++s) x[s] = *reinterpret_cast<const f32x4_t*>(p + (size_t)s * stride);
#pragma unroll
  for (int s = 0; s < S; ++s) v += x[s];
  return v;
}

// PACKED 1: only the first *live rows are there; 2: row m of xn comes from row live[m], or is zero (back to block rows).
template <typename T, int S, int PACKED>
__global__ __launch_bounds__(1024) void k_residual_norm(float* __restrict__ h, const float* __restrict__ part,
                                                        size_t split_stride, int d, const T* __restrict__ gain,
                                                        float eps, T* __restrict__ xn, const int32_t* __restrict__ live) {
  __shared__ float red[16];
  d = with_args(d, h, part, split_stride, gain, eps, xn, live, __builtin_amdgcn_workgroup_size_x());
  const size_t row_out = blockIdx.x;
  const int d4 = d >> 2, tid = threadIdx.x, step = blockDim.x;
  size_t row = row_out;
  if (PACKED == 1 && (int)row >= *live) return;
  if (PACKED == 2) {
    const int at = live[row_out];
    if (at < 0) {
      const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
      for (int i = tid; i < d4; i += step) Pack4<T>::store(xn + row_out * d + 4 * i, zero);
      return;
    }
    row = (size_t)at;
  }
  float* hr = h + row * d;
  f32x4_t keep = {0.f, 0.f, 0.f, 0.f};               // this thread's first column
  typename Pack4<T>::Raw g0 = {};                    // and its gain, as it was loaded: converting it here would wait for it
  if (tid < d4) g0 = *reinterpret_cast<const typename Pack4<T>::Raw*>(gain + 4 * tid);
  float ss = 0.f;
  for (int i = tid; i < d4; i += step) {
    const f32x4_t v = add_splits<S>(*reinterpret_cast<const f32x4_t*>(hr + 4 * i), part + row * d + 4 * i, split_stride);
    *reinterpret_cast<f32x4_t*>(hr + 4 * i) = v;
    if (i == tid) keep = v;
    ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
  }
  const float inv = rms_scale(ss, d, eps, red);
  for (int i = tid; i < d4; i += step) {
    const f32x4_t v = i == tid ? keep : *reinterpret_cast<const f32x4_t*>(hr + 4 * i);   // written by this thread above
    const f32x4_t g = i == tid ? Pack4<T>::value(g0) : Pack4<T>::load(gain + 4 * i);
    Pack4<T>::store(xn + row_out * d + 4 * i, v * inv * g);
  }
}

// the split count of a launch as a template argument (gemm_plan gives at most 8)
#define ESP_SPLITS(splits, ...)                                   \
  switch (splits) {                                               \
    case 1: { constexpr int S = 1; __VA_ARGS__; } break;          \
    case 2: { constexpr int S = 2; __VA_ARGS__; } break;          \
    case 3: { constexpr int S = 3; __VA_ARGS__; } break;          \
    case 4: { constexpr int S = 4; __VA_ARGS__; } break;          \
    case 5: { constexpr int S = 5; __VA_ARGS__; } break;          \
    case 6: { constexpr int S = 6; __VA_ARGS__; } break;          \
    case 7: { constexpr int S = 7; __VA_ARGS__; } break;          \
    case 8: { constexpr int S = 8; __VA_ARGS__; } break;          \
    default: return hipErrorInvalidValue;                         \
  }

hipError_t launch_residual_norm(hipStream_t st, int dtype, float* h, const float* part, int splits, int M,
                                int d, const void* gain, float eps, void* xn_out, const int32_t* n_live,
                                const int32_t* packed_row) {
  const dim3 grid(M), block(norm_threads(d));
  const size_t stride = (size_t)M * d;
#define ESP_NORM(T_, S_, P_, LIVE_)                                                                                      \
  hipLaunchKernelGGL((k_residual_norm<T_, S_, P_>), grid, block, 0, st, h, part, stride, d, (const T_*)gain, eps, (T_*)xn_out, \
                     (const int32_t*)(LIVE_))
  if (dtype == ESP_F32) {          // the fp32 GEMM splits K inside a workgroup; fp32 batches are not packed
    if (splits != 1 || n_live || packed_row) return hipErrorInvalidValue;
    ESP_NORM(float, 1, 0, nullptr);
  } else if (packed_row) {
    ESP_SPLITS(splits, ESP_NORM(bf16_t, S, 2, packed_row));
  } else if (n_live) {
    ESP_SPLITS(splits, ESP_NORM(bf16_t, S, 1, n_live));
  } else {
    ESP_SPLITS(splits, ESP_NORM(bf16_t, S, 0, nullptr));
  }
#undef ESP_NORM
  return hipGetLastError();
}

// ---- QKV epilogue: split-K reduce, optional per-head RMSNorm, rotary, KV append ----------------
// hd/8 lanes per (row, head): a lane owns the features 4 i .. 4 i + 3 of both halves of the head, i.e. four
// rotary pairs, as two 16-byte pieces of every partial; all 2 S loads are in flight at once.
template <typename T, int HD, int S, bool PACKED>
__global__ __launch_bounds__(256) void k_qkv_post(BlockDev b, KvDev kv, int layer, const float* __restrict__ part,
                                                  size_t split_stride, int hq, int hkv, int qk_norm,
                                                  const T* __restrict__ qg, const T* __restrict__ kg, float eps,
                                                  const float* __restrict__ rope_tab, T* __restrict__ q_out) {
  constexpr int LPH = HD / 8, HALF = HD / 2;
  hq = with_args(hq, part, split_stride, rope_tab, q_out, kv.len, kv.base, kv.seq_cap, kv.capacity);
  hq = with_args(hq, b.n_rows, b.rows_per_seq, kv.len_bound, kv.k, kv.v, layer, hkv, qk_norm);
  const int row = blockIdx.y;                       // of the activations
  if (PACKED && row >= *b.n_live()) return;
  const int hidx = (blockIdx.x * 256 + threadIdx.x) / LPH;
  const int f0 = (threadIdx.x % LPH) * 4;
  const int n_heads = hq + 2 * hkv;
  if (hidx >= n_heads) return;
  // The sequence's scalars, the partials and the rotary table's entries (a row of it for every row of the activations), all asked for
  // before the first of them is waited for: 68 rows of 32 + 16 heads 5.1 -> 4.8 us.
  const int brow = PACKED ? b.live_rows()[row] : row;
  const int seq = (int)((unsigned)brow / (unsigned)b.rows_per_seq), r = brow - seq * b.rows_per_seq;
  const int nr = b.n_rows[seq], base = kv.base[seq], len = kv.len[seq], cap = kv.seq_cap[seq];
  __builtin_amdgcn_sched_barrier(0);
  const size_t c0 = ((size_t)row * n_heads + hidx) * HD + f0;
  const float* rt = rope_tab + ((size_t)row * HALF + f0) * 2;      // cos, sin of four pairs
  f32x4_t t0 = *reinterpret_cast<const f32x4_t*>(rt), t1 = *reinterpret_cast<const f32x4_t*>(rt + 4);
  f32x4_t p0[S], p1[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    p0[s] = *reinterpret_cast<const f32x4_t*>(part + c0 + (size_t)s * split_stride);
    p1[s] = *reinterpret_cast<const f32x4_t*>(part + c0 + (size_t)s * split_stride + HALF);
  }
  __builtin_amdgcn_sched_barrier(0);
  const bool live = seq_valid(kv, len, base, cap, nr) && nr <= b.rows_per_seq && r < nr;
  const int64_t slot = (int64_t)(uint32_t)base + (uint32_t)len + r;   // of a live row: none is negative
  f32x4_t x0 = {0.f, 0.f, 0.f, 0.f}, x1 = x0;            // added in split order
#pragma unroll
  for (int s = 0; s < S; ++s) { x0 += p0[s]; x1 += p1[s]; }
  asm volatile("" : "+v"(t0), "+v"(t1));                 // here, not in the branch that uses them
  if (hidx < hq + hkv) {
    if (qk_norm) {
      // The squares are added as a balanced tree over the rotary pairs, the farthest pairs first (distance
      // HD/4, HD/8, ..., 1): across the lanes for each of the four pairs, then the pairs of the lane.  Order and
      // fused form fix the last bit of the norm, which a bf16 model carries through its layers.
      float sq[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) sq[e] = fmaf(x1[e], x1[e], x0[e] * x0[e]);
#pragma unroll
      for (int o = LPH / 2; o > 0; o >>= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) sq[e] += __shfl_xor(sq[e], o, 64);
      const float ss = (sq[0] + sq[2]) + (sq[1] + sq[3]);
      const float inv = 1.0f / sqrtf(ss / (float)HD + eps);
      const T* g = (hidx < hq ? qg : kg) + f0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {   // scalar loads: the caller's gains need no more than their type's alignment
        x0[e] *= inv * to_f32(g[e]);
        x1[e] *= inv * to_f32(g[HALF + e]);
      }
    }
    const f32x4_t c = {t0[0], t0[2], t1[0], t1[2]}, s = {t0[1], t0[3], t1[1], t1[3]};
    const f32x4_t y0 = x0 * c - x1 * s, y1 = x1 * c + x0 * s;
    if (hidx < hq) {   // a row that is not there: its query is zero, whatever its partials hold
      T* qo = q_out + ((size_t)row * hq + hidx) * HD + f0;
      const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
      Pack4<T>::store(qo, live ? y0 : zero);
      Pack4<T>::store(qo + HALF, live ? y1 : zero);
    } else if (live) {       // four features are consecutive in a K fragment
      T* kp = (T*)kv.k + kv_plane(layer, hidx - hq, hkv, kv.capacity, HD);
      if constexpr (HD == 128 && sizeof(T) == 2) {   // the attention kernel of this form reads 16-byte pieces anyway
        Pack4<T>::store(kp + k_off(slot, f0, HD), y0);
        Pack4<T>::store(kp + k_off(slot, f0 + HALF, HD), y1);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          kp[k_off(slot, f0 + e, HD)] = from_f32<T>(y0[e]);
          kp[k_off(slot, f0 + HALF + e, HD)] = from_f32<T>(y1[e]);
        }
      }
    }
  } else if (live) {
    T* vp = (T*)kv.v + kv_plane(layer, hidx - hq - hkv, hkv, kv.capacity, HD);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      vp[v_off(slot, f0 + e, HD)] = from_f32<T>(x0[e]);
      vp[v_off(slot, f0 + HALF + e, HD)] = from_f32<T>(x1[e]);
    }
  }
}

hipError_t launch_qkv_post(hipStream_t st, int dtype, const BlockDev& b, const KvDev& kv, int layer,
                           const float* part, int splits, int M, int hq, int hkv, int hd, int qk_norm,
                           const void* qg, const void* kg, float eps, const float* rope_tab, void* q_out) {
  const int n_heads = hq + 2 * hkv;
  const dim3 grid((n_heads * (hd / 8) + 255) / 256, M);
  const size_t stride = (size_t)M * n_heads * hd;
#define ESP_QKV_POST(T_, HD_, S_, P_)                                                                                     \
  hipLaunchKernelGGL((k_qkv_post<T_, HD_, S_, P_>), grid, dim3(256), 0, st, b, kv, layer, part, stride, hq, hkv, qk_norm, \
                     (const T_*)qg, (const T_*)kg, eps, rope_tab, (T_*)q_out)
  if (dtype == ESP_F32) {
    if (splits != 1) return hipErrorInvalidValue;
    if (hd == 64) ESP_QKV_POST(float, 64, 1, false);
    else ESP_QKV_POST(float, 128, 1, false);
  } else if (hd == 64) {
    if (b.packed) { ESP_SPLITS(splits, ESP_QKV_POST(bf16_t, 64, S, true)); }
    else { ESP_SPLITS(splits, ESP_QKV_POST(bf16_t, 64, S, false)); }
  } else {
    if (b.packed) { ESP_SPLITS(splits, ESP_QKV_POST(bf16_t, 128, S, true)); }
    else { ESP_SPLITS(splits, ESP_QKV_POST(bf16_t, 128, S, false)); }
  }
#undef ESP_QKV_POST
  return hipGetLastError();
}

// ---- argmax over the vocabulary, lowest id on ties ------------------------------------------------
__global__ __launch_bounds__(256) void k_argmax(const float* __restrict__ logits, size_t row_stride,
                                                const int32_t* __restrict__ row_map, int vocab,
                                                int32_t* __restrict__ out, const int32_t* __restrict__ out_index,
                                                const int32_t* __restrict__ draw_pos, uint32_t seed) {
  __shared__ float sv[4];
  __shared__ int si[4];
  const int m = blockIdx.x;
  const int dst = out_index ? out_index[m] : m;
  if (dst < 0) return;
  const size_t src = row_map ? (size_t)row_map[m] : (size_t)m;
  const float* p = logits + src * row_stride;
  const bool draw = draw_pos != nullptr;
  const uint32_t pos = draw ? (uint32_t)draw_pos[m] : 0u;
  float best = -INFINITY;
  int bi = 0x7fffffff;
  // eight loads in flight: 4096 logits a row, 15 rows: 7.2 -> 4.1 us
  constexpr int U = 8;
  for (int i0 = threadIdx.x; i0 < vocab; i0 += 256 * U) {
    float x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = i0 + 256 * u < vocab ? p[i0 + 256 * u] : -INFINITY;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + 256 * u;
      const float v = draw ? x[u] + gumbel_noise(seed, pos, (uint32_t)i) : x[u];
      if (v > best) { best = v; bi = i; }   // ascending i per thread: first maximum is kept
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    float ov = __shfl_xor(best, o, 64);
    int oi = __shfl_xor(bi, o, 64);
    if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
  }
  if ((threadIdx.x & 63) == 0) { sv[threadIdx.x >> 6] = best; si[threadIdx.x >> 6] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w)
      if (sv[w] > best || (sv[w] == best && si[w] < bi)) { best = sv[w]; bi = si[w]; }
    out[dst] = bi == 0x7fffffff ? 0 : bi;
  }
}

hipError_t launch_argmax(hipStream_t st, const float* logits, size_t row_stride, const int32_t* row_map,
                         int n_rows_out, int vocab, int32_t* out, const int32_t* out_index,
                         const int32_t* draw_pos, uint32_t seed) {
  if (n_rows_out <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_argmax, dim3(n_rows_out), dim3(256), 0, st, logits, row_stride, row_map, vocab, out,
                     out_index, draw_pos, seed);
  return hipGetLastError();
}

// ---- plain rows <-> cache layout --------------------------------------------------------------------
template <typename T>
__global__ void k_kv_copy(KvDev kv, int layer, int n_kv, int hd, int seq_base, int first_slot, int n_slots,
                          T* k_rows, T* v_rows, int to_cache) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t total = (size_t)n_slots * n_kv * hd;
  if (i >= total) return;
  int d = (int)(i % hd);
  int kvh = (int)((i / hd) % n_kv);
  int s = (int)(i / ((size_t)hd * n_kv));
  int64_t slot = (int64_t)seq_base + first_slot + s;
  T* kp = (T*)kv.k + kv_plane(layer, kvh, n_kv, kv.capacity, hd);
  T* vp = (T*)kv.v + kv_plane(layer, kvh, n_kv, kv.capacity, hd);
  if (to_cache) {
    kp[k_off(slot, d, hd)] = k_rows[i];
    vp[v_off(slot, d, hd)] = v_rows[i];
  } else {
    k_rows[i] = kp[k_off(slot, d, hd)];
    v_rows[i] = vp[v_off(slot, d, hd)];
  }
}

hipError_t launch_kv_copy(hipStream_t st, int dtype, const KvDev& kv, int layer, int n_kv, int hd, int seq_base,
                          int first_slot, int n_slots, void* k_rows, void* v_rows, int to_cache) {
  size_t total = (size_t)n_slots * n_kv * hd;
  if (total == 0) return hipSuccess;
  ESP_DISPATCH(dtype, hipLaunchKernelGGL(k_kv_copy<T>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                                         kv, layer, n_kv, hd, seq_base, first_slot, n_slots, (T*)k_rows,
                                         (T*)v_rows, to_cache));
  return hipGetLastError();
}

// ---- mask vectors (Sec. 3.1 Eq. 4 and Eq. 5) -----------------------------------------------------------
// Mean of the prompt's token embeddings.  A workgroup owns 64 features: 16 lanes of four features side by side (a
// 128-byte line of a bf16 row) times 64 groups of tokens, each with eight rows in flight, added up through LDS in group
// order.  The time is that of the gather: 2049 tokens of d = 4096 took 896 us with a thread per feature walking all tokens.
// VEC: rows start at a multiple of the four features' size.
constexpr int MEAN_GROUPS = 64, MEAN_U = 8;
template <typename T, bool VEC>
__global__ __launch_bounds__(1024) void k_mask_mean(const T* __restrict__ embed, const int32_t* __restrict__ tokens, int n, int k,
                                                    int d, int vocab, T* __restrict__ mask_embed) {
  __shared__ f32x4_t part[MEAN_GROUPS][16];
  const int lane = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int i = blockIdx.x * 64 + lane * 4;          // d is a multiple of 4
  const bool in = i < d;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  for (int t0 = grp; t0 < n; t0 += MEAN_GROUPS * MEAN_U) {
    int id[MEAN_U];
#pragma unroll
    for (int u = 0; u < MEAN_U; ++u) {
      const int t = t0 + u * MEAN_GROUPS;
      id[u] = t < n ? tokens[t] : -1;
    }
    f32x4_t x[MEAN_U];
#pragma unroll
    for (int u = 0; u < MEAN_U; ++u) {
      x[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      if (in && id[u] >= 0 && id[u] < vocab) {
        const T* row = embed + (size_t)id[u] * d + i;
        if constexpr (VEC) {
          x[u] = Pack4<T>::load(row);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) x[u][e] = to_f32(row[e]);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < MEAN_U; ++u) acc += x[u];
  }
  part[grp][lane] = acc;
  __syncthreads();
  if (grp != 0 || !in) return;
  f32x4_t sum = part[0][lane];
  for (int g = 1; g < MEAN_GROUPS; ++g) sum += part[g][lane];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const T v = from_f32<T>(sum[e] / (float)n);
    for (int j = 0; j < k; ++j) mask_embed[(size_t)j * d + i + e] = v;
  }
}

hipError_t launch_mask_mean(hipStream_t st, int dtype, const void* embed, const int32_t* tokens, int n, int k,
                            int d, int vocab, void* mask_embed) {
  ESP_DISPATCH(dtype, {
    const bool vec = (uintptr_t)embed % (4 * sizeof(T)) == 0;
    hipLaunchKernelGGL((vec ? k_mask_mean<T, true> : k_mask_mean<T, false>), dim3((d + 63) / 64), dim3(1024), 0, st,
                       (const T*)embed, tokens, n, k, d, vocab, (T*)mask_embed);
  });
  return hipGetLastError();
}

// Hard initialisation (Sec. 4, mask-design variant a): mask i = embedding of the prompt token
// k - i places before the end.
template <typename T>
__global__ void k_mask_last_k(const T* __restrict__ embed, const int32_t* __restrict__ tokens, int n, int k, int d,
                              int vocab, T* __restrict__ mask_embed) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d) return;
  for (int j = 0; j < k; ++j) {
    int id = tokens[n - k + j];
    mask_embed[(size_t)j * d + i] = id >= 0 && id < vocab ? embed[(size_t)id * d + i] : from_f32<T>(0.f);
  }
}

hipError_t launch_mask_last_k(hipStream_t st, int dtype, const void* embed, const int32_t* tokens, int n, int k,
                              int d, int vocab, void* mask_embed) {
  ESP_DISPATCH(dtype, hipLaunchKernelGGL(k_mask_last_k<T>, dim3((d + 255) / 256), dim3(256), 0, st, (const T*)embed,
                                         tokens, n, k, d, vocab, (T*)mask_embed));
  return hipGetLastError();
}

// Gaussian fit to the embedding table (Sec. 4, variant b): mu[i] = mean over the vocabulary of
// column i, sigma = root mean square deviation of all entries from their column's mean.  Two
// passes over the table (mean, then squared deviations), each split into slabs of rows whose
// fp32 partial sums are added up in fp64, in slab order.
// MODE 0: partial[slab][i] = sum of column i over the slab; 1: sum of (x - mu[i])^2
template <typename T, int MODE>
__global__ __launch_bounds__(256) void k_embed_stats_partial(const T* __restrict__ embed, int vocab, int d,
                                                             int rows_per_slab, const float* __restrict__ mu,
                                                             float* __restrict__ partial) {
  const int i = blockIdx.x * 256 + threadIdx.x, slab = blockIdx.y;
  if (i >= d) return;
  const int v0 = slab * rows_per_slab, v1 = min(vocab, v0 + rows_per_slab);
  const float c = MODE ? mu[i] : 0.f;
  float acc = 0.f;
  for (int v = v0; v < v1; ++v) {
    const float x = to_f32(embed[(size_t)v * d + i]) - c;
    acc += MODE ? x * x : x;
  }
  partial[(size_t)slab * d + i] = acc;
}

__global__ __launch_bounds__(256) void k_embed_mean_final(const float* __restrict__ partial, int slabs, int d, int vocab,
                                                          float* __restrict__ mu) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= d) return;
  double s = 0.0;
  for (int b = 0; b < slabs; ++b) s += (double)partial[(size_t)b * d + i];
  mu[i] = (float)(s / (double)vocab);
}

// one workgroup: sigma = sqrt(sum of all partials / (vocab * d))
__global__ __launch_bounds__(256) void k_embed_sigma_final(const float* __restrict__ partial, int slabs, int d, int vocab,
                                                           float* __restrict__ sigma) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < d; i += 256)
    for (int b = 0; b < slabs; ++b) s += (double)partial[(size_t)b * d + i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) sigma[0] = (float)sqrt(red[0] / ((double)vocab * (double)d));
}

// m_j = mu + (shift + z_j) sigma; z: [k][d] standard normal draws of the caller, or null
template <typename T>
__global__ void k_mask_affine(const float* __restrict__ mu, const float* __restrict__ sigma,
                              const float* __restrict__ z, float shift, int k, int d, T* __restrict__ mask_embed) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d) return;
  const float sg = sigma[0], m = mu[i];
  for (int j = 0; j < k; ++j)
    mask_embed[(size_t)j * d + i] = from_f32<T>(fmaf(shift + (z ? z[(size_t)j * d + i] : 0.f), sg, m));
}

size_t mask_gaussian_scratch_floats(int d) { return (size_t)2 * d + 64; }   // least: one slab

hipError_t launch_mask_gaussian(hipStream_t st, int dtype, const void* embed, int vocab, int d, const float* z,
                                float shift, int k, float* scratch, size_t scratch_floats, void* mask_embed) {
  // scratch: mu [d], sigma [64 (one used)], partial [slabs][d]
  float* mu = scratch;
  float* sigma = scratch + d;
  float* partial = scratch + d + 64;
  const size_t room = (scratch_floats - d - 64) / d;
  const int slabs = (int)std::max<size_t>(1, std::min<size_t>(room, 256));
  const int rows_per_slab = (vocab + slabs - 1) / slabs;
  const int used = (vocab + rows_per_slab - 1) / rows_per_slab;
  const dim3 grid((d + 255) / 256, used);
  ESP_DISPATCH(dtype, hipLaunchKernelGGL((k_embed_stats_partial<T, 0>), grid, dim3(256), 0, st, (const T*)embed, vocab,
                                         d, rows_per_slab, (const float*)nullptr, partial));
  hipLaunchKernelGGL(k_embed_mean_final, dim3((d + 255) / 256), dim3(256), 0, st, partial, used, d, vocab, mu);
  ESP_DISPATCH(dtype, hipLaunchKernelGGL((k_embed_stats_partial<T, 1>), grid, dim3(256), 0, st, (const T*)embed, vocab,
                                         d, rows_per_slab, (const float*)mu, partial));
  hipLaunchKernelGGL(k_embed_sigma_final, dim3(1), dim3(256), 0, st, partial, used, d, vocab, sigma);
  ESP_DISPATCH(dtype, hipLaunchKernelGGL(k_mask_affine<T>, dim3((d + 255) / 256), dim3(256), 0, st, mu, sigma, z, shift,
                                         k, d, (T*)mask_embed));
  return hipGetLastError();
}

template <typename T>
__global__ void k_mask_ema(const T* __restrict__ embed, const int32_t* __restrict__ n_emit,
                           const int32_t* __restrict__ emit_tok, float lambda, int k, int d, int vocab,
                           T* __restrict__ mask_embed) {
  // blockIdx.y: the sequence whose vectors ([k, d] at mask_embed + y * k * d) follow its own last
  // emitted token; a launch with one row of workgroups updates the shared vectors from sequence 0
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d) return;
  const int seq = blockIdx.y;
  int ne = n_emit[seq];
  if (ne < 1 || ne > ESP_MAX_MASKS + 1) return;
  int id = emit_tok[(size_t)seq * (ESP_MAX_MASKS + 1) + ne - 1];
  if (id < 0 || id >= vocab) return;
  float e = to_f32(embed[(size_t)id * d + i]);
  T* me = mask_embed + (size_t)seq * k * d;
  for (int j = 0; j < k; ++j) {
    float m = to_f32(me[(size_t)j * d + i]);
    me[(size_t)j * d + i] = from_f32<T>(m + lambda * (e - m));
  }
}

hipError_t launch_mask_ema(hipStream_t st, int dtype, const void* embed, const int32_t* n_emit,
                           const int32_t* emit_tok, float lambda, int k, int d, int vocab, void* mask_embed,
                           int n_seq) {
  ESP_DISPATCH(dtype, hipLaunchKernelGGL(k_mask_ema<T>, dim3((d + 255) / 256, n_seq), dim3(256), 0, st, (const T*)embed,
                                         n_emit, emit_tok, lambda, k, d, vocab, (T*)mask_embed));
  return hipGetLastError();
}
