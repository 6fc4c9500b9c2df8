// Tree-masked grouped-query attention of one decoder layer (paper Sec. 3.3, App. C, App. E).
//
// Row r of sequence b attends to cache slots [0, len[b]) and to the block rows c whose bit is set
// in its ancestor bitset (held at slots len[b] + c).  Only the last n_rows keys of a sequence need
// a mask test; every tile that lies inside the committed cache runs unmasked.
//
// bf16 / head_dim 128 path (k_attn_ring, described at its definition): the G = n_q/n_kv query heads
// of a kv head times the block rows form the "query columns" of a (keys x queries) problem; a
// workgroup owns the columns of one kv head and one split of the key range, and the per-split partial
// (m, l, O) are merged by k_attn_merge_ring in split order (fixed, so results do not depend on
// scheduling).
//
// Generic path (k_attn_generic): one wave per (row, head, split), any dtype / head_dim multiple of
// 64; used by the fp32 tiny configuration.
#include <algorithm>
#include <type_traits>

#include "esp_internal.h"

namespace {

constexpr float LOG2E = 1.4426950408889634f;
constexpr float NEG_BIG = -1.0e30f;

// one condition after the other (k_attn_generic says where)
__device__ __forceinline__ bool seq_ok_in_turn(const KvDev& kv, int seq, int n_rows, int rows_per_seq) {
  const int L = kv.len[seq], base = kv.base[seq], cap = kv.seq_cap[seq];
  return L >= 0 && L <= kv.len_bound && n_rows >= 0 && n_rows <= rows_per_seq && L + n_rows <= cap && base >= 0 && (base & 63) == 0 &&
         (int64_t)base + cap <= kv.capacity;
}
// UNIFORM: seq is the same for the wave, in a scalar
template <bool UNIFORM = false>
__device__ __forceinline__ bool seq_ok(const KvDev& kv, int seq, int n_rows, int rows_per_seq) {
  const int base = kv.base[seq], cap = kv.seq_cap[seq];
  int L = kv.len[seq];
  if (UNIFORM) L = with_args(L, base, cap, n_rows, kv.len_bound);   // the loads together, and no short circuit
  return (L >= 0) & (L <= kv.len_bound) & (n_rows >= 0) & (n_rows <= rows_per_seq) & (L + n_rows <= cap) & (base >= 0) &
         ((base & 63) == 0) & ((int64_t)base + cap <= kv.capacity);
}

// --------------------------------------------------------------------------------------------------
// eight consecutive elements of the cache (one 16-byte or two) as floats; VEC: the planes are 16-byte aligned
template <bool VEC, typename T>
__device__ __forceinline__ void load8(const T* p, float (&v)[8]) {
  if constexpr (VEC && sizeof(T) == 4) {
    const f32x4_t a = *reinterpret_cast<const f32x4_t*>(p), b = *reinterpret_cast<const f32x4_t*>(p + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
  } else if constexpr (VEC) {
    const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(p);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (float)a[e];
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = to_f32(p[e]);
  }
}

// LDS traffic inside one wave (its operations are done in order): the compiler keeps the order
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wave per (row, head, split); a lane has one key of a tile for the scores and HD / 64 features for the output.  The
// tile's K and V sit in fragment order, eight features of a key or eight keys of a feature side by side: all of them are
// in flight before the first is used (a load an element was 14.5 us at 60 rows and 188 keys, and with them one split of
// three tiles; now 5.6 in three splits).  Sums run over features and keys in ascending order.
// MERGE: the splits of a (row, head) are waves of one workgroup, up to MERGE of them, which merge through LDS in split order (as
// k_attn_merge does from memory) and write the result: a launch less, 60 rows on 128 keys 5.6 + 4.3 -> 6.1 us.
// Three waves a SIMD of HD 64 (two took 170 registers where three have 168: 400 rows on 16 keys 20.8 -> 22.7 us).
template <typename T, int HD, bool PACKED, bool VEC, int MERGE>
__global__ __launch_bounds__(64 * (MERGE ? MERGE : 1), HD == 64 ? 3 : 1) void k_attn_generic(BlockDev b, KvDev kv, int layer, int hq, int hkv,
                                                                          const T* __restrict__ q, float* __restrict__ part_o,
                                                                          float* __restrict__ part_ml, int nsplit, int tps,
                                                                          T* __restrict__ out) {
  constexpr int WAVES = MERGE ? MERGE : 1;
  __shared__ float qs_w[WAVES][HD];
  __shared__ float ps_w[WAVES][64];
  __shared__ float m_w[WAVES], l_w[WAVES];
  auto sync = [] { if constexpr (MERGE > 0) wave_sync(); else __syncthreads(); };
  const int row = blockIdx.x, h = blockIdx.y, lane = MERGE ? threadIdx.x & 63 : threadIdx.x;
  const int wave = MERGE ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0, sp = MERGE ? wave : (int)blockIdx.z;
  float* qs = qs_w[wave];
  float* ps = ps_w[wave];
  const int seq = row / b.rows_per_seq, r = row % b.rows_per_seq;
  const int nr = b.n_rows[seq];
  // What the compiler makes of the key loop depends on how it comes by these scalars: fp32 with HD 64 takes 0.92 to 0.98 of the time with
  // one condition after the other, bf16 1.05 to 1.1 and HD 128 1.03 to 1.07 (20 rows on 16000 keys, four sequences 164 -> 151 us, 339 -> 368,
  // 315 -> 330).
  const bool ok = sizeof(T) == 4 && HD == 64 ? seq_ok_in_turn(kv, seq, nr, b.rows_per_seq) : seq_ok<(MERGE > 0)>(kv, seq, nr, b.rows_per_seq);
  if (!ok || r >= nr) {
    if (MERGE && !PACKED)
      for (int d = threadIdx.x; d < HD; d += blockDim.x) out[((size_t)row * hq + h) * HD + d] = from_f32<T>(0.f);
    return;
  }
  const int L = kv.len[seq], total = L + nr;
  const int ntiles = (total + 63) >> 6;
  const int t0 = sp * tps, t1 = min(ntiles, t0 + tps);
  const int kvh = h / (hq / hkv);
  const T* kp = (const T*)kv.k + kv_plane(layer, kvh, hkv, kv.capacity, HD);
  const T* vp = (const T*)kv.v + kv_plane(layer, kvh, hkv, kv.capacity, HD);
  const int64_t base = kv.base[seq];
  const float scale = LOG2E / sqrtf((float)HD);
  for (int d = lane; d < HD; d += 64) qs[d] = to_f32(q[(act_row<PACKED>(b, seq, r) * hq + h) * HD + d]) * scale;
  sync();
  const uint64_t* anc = b.anc + (size_t)row * b.anc_words;
  float m = NEG_BIG, l = 0.f;
  float o[HD / 64];
#pragma unroll
  for (int i = 0; i < HD / 64; ++i) o[i] = 0.f;
  for (int t = t0; t < t1; ++t) {
    const int key = t * 64 + lane;
    bool valid = key < total;
    float kf[HD / 8][8];
    if (valid) {
#pragma unroll
      for (int g = 0; g < HD / 8; ++g) load8<VEC>(kp + k_off(base + key, 8 * g, HD), kf[g]);
    }
    float vf[HD / 64][8][8];                    // [.][piece: block, step, half][key 8 (e / 4) + e % 4 of it]
#pragma unroll
    for (int i = 0; i < HD / 64; ++i)
#pragma unroll
      for (int c = 0; c < 8; ++c)               // (the whole tile lies inside the plane: sequences own 64-aligned slots)
        load8<VEC>(vp + v_off(base + t * 64 + (c >> 2) * 32 + ((c >> 1) & 1) * 16 + (c & 1) * 4, lane + 64 * i, HD), vf[i][c]);
    if (valid && key >= L) {
      int c = key - L;
      valid = (anc[c >> 6] >> (c & 63)) & 1ull;
    }
    float s = NEG_BIG;
    if (valid) {
      float acc = 0.f;
#pragma unroll
      for (int d = 0; d < HD; ++d) acc = fmaf(kf[d >> 3][d & 7], qs[d], acc);
      s = acc;
    }
    float m_new = fmaxf(m, wave_max(s));
    float p = valid ? exp2f(s - m_new) : 0.f;
    float alpha = exp2f(m - m_new);
    l = l * alpha + wave_sum(p);
    m = m_new;
    ps[lane] = p;
    sync();
    const int nk = min(64, total - t * 64);     // entries past the sequence are not touched: cache memory may hold anything
#pragma unroll
    for (int i = 0; i < HD / 64; ++i) {
      float a = o[i] * alpha;
#pragma unroll
      for (int kk = 0; kk < 64; ++kk) {
        const int c = (kk >> 5) * 4 + ((kk >> 4) & 1) * 2 + ((kk >> 2) & 1), e = ((kk >> 3) & 1) * 4 + (kk & 3);
        a = fmaf(ps[kk], kk < nk ? vf[i][c][e] : 0.f, a);
      }
      o[i] = a;
    }
    sync();
  }
  if constexpr (MERGE > 0) {
    if (lane == 0) { m_w[wave] = m; l_w[wave] = l; }
#pragma unroll
    for (int i = 0; i < HD / 64; ++i) qs[lane + 64 * i] = o[i];        // the query is done with
    __syncthreads();
    T* dst = out + (act_row<PACKED>(b, seq, r) * hq + h) * HD;
    for (int d = threadIdx.x; d < HD; d += blockDim.x) {
      float mx = NEG_BIG;
      for (int s = 0; s < nsplit; ++s) mx = fmaxf(mx, m_w[s]);
      float lt = 0.f, acc = 0.f;
      for (int s = 0; s < nsplit; ++s) {
        const float w = exp2f(m_w[s] - mx);
        lt += l_w[s] * w;
        acc += qs_w[s][d] * w;
      }
      const float inv = lt > 0.f ? 1.f / lt : 0.f;
      dst[d] = from_f32<T>(acc * inv);
    }
    return;
  }
  const size_t item = ((size_t)row * hq + h) * nsplit + sp;
#pragma unroll
  for (int i = 0; i < HD / 64; ++i) part_o[item * HD + lane + 64 * i] = o[i];
  if (lane == 0) {
    part_ml[item * 2 + 0] = m;
    part_ml[item * 2 + 1] = l;
  }
}

// --------------------------------------------------------------------------------------------------
// k_attn_ring: the bf16 / head_dim 128 kernel.
//
// One workgroup per CU owns up to 384 query columns (query row x head of one kv group; a wave per
// 32 columns, 4 to 12 waves, so two to three waves share a SIMD and the softmax arithmetic of one
// overlaps the matrix work of another) and one split of the key range.  K/V tiles of 64 keys
// (16 KB + 16 KB, already in fragment order in the cache) go from global memory straight into a
// ring of four LDS stages (no register hop, up to three tiles in flight) and are shared by all the
// waves.  S^T = K Q^T and O^T = V^T P^T both run on v_mfma_f32_32x32x16_bf16: computing the
// transposed scores leaves each lane with one query column and 16 keys per 32-key block, which is
// exactly the B-operand layout P^T needs, so the probabilities never leave registers.  Online
// softmax in fp32 (base-2 exponent), one exchange between the two lane halves per 32 keys.
// Partial (m, l, O) per split are merged by k_attn_merge_ring in split order (fixed, so results do
// not depend on scheduling).
constexpr int K_TILE_BYTES = 64 * 128 * 2;   // 64 keys: two cache blocks of 32 slots, 16 fragments of 1 KB
constexpr int V_TILE_BYTES = 64 * 128 * 2;
constexpr int RING_STAGES = 4;
constexpr int STAGE_BYTES = K_TILE_BYTES + V_TILE_BYTES;
constexpr int RING_LDS_BYTES = RING_STAGES * STAGE_BYTES;
constexpr int RING_MAX_WAVES = 12;
// The reference m of a column's exponents follows its running maximum lazily: it is set by the first
// unit that has a visible key and moves only when a score exceeds it by more than this many powers of
// two, so the output accumulators are rescaled a few times per split instead of at almost every unit.
// Probabilities may reach 2^RESCALE_SLACK, which fp32 sums and the bf16 operand of the P V product
// hold without loss of relative precision.
constexpr float RESCALE_SLACK = 24.0f;

// Visibility bits of 64 consecutive keys for one block row: bit j stands for block position
// c_lo + j (negative positions are committed cache slots, always visible; positions from
// keys_in_tile on lie past the sequence).  anc is the row's ancestor bitset.
__device__ __forceinline__ uint64_t key_window(const uint64_t* __restrict__ anc, int anc_words, int c_lo,
                                               int keys_in_tile) {
  uint64_t wnd;
  if (c_lo < 0) {
    const int n = -c_lo;                                   // 1..63 cache keys lead the tile
    const uint64_t a0 = anc_words > 0 ? anc[0] : 0ull;
    wnd = (a0 << n) | ((1ull << n) - 1ull);
  } else {
    const int w0 = c_lo >> 6, sh = c_lo & 63;
    const uint64_t a0 = w0 < anc_words ? anc[w0] : 0ull;
    const uint64_t a1 = w0 + 1 < anc_words ? anc[w0 + 1] : 0ull;
    wnd = sh ? (a0 >> sh) | (a1 << (64 - sh)) : a0;
  }
  if (keys_in_tile < 64) wnd &= (1ull << keys_in_tile) - 1ull;
  return wnd;
}

// zeroes, in the LDS copy of the sequence's last tile, the V entries of keys past its end (their
// probability is zero, but 0 * NaN from never-written cache memory would poison the accumulators)
__device__ __forceinline__ void ring_zero_tail(unsigned char* vs, int keys_left, int tid, int nthreads) {
  for (int p = tid; p < 1024; p += nthreads) {
    u32x4_t v = *reinterpret_cast<u32x4_t*>(vs + p * 16);
    // piece p = fragment (block p/512, key-step (p/64)%2) of lane p%64; word w holds elements
    // 2w, 2w+1 = keys k0, k0+1
    const int kbase = (p >> 9) * 32 + ((p >> 6) & 1) * 16 + ((p >> 5) & 1) * 4;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int k0 = kbase + 8 * (w >> 1) + 2 * (w & 1);
      v[w] &= k0 + 1 < keys_left ? 0xffffffffu : (k0 < keys_left ? 0x0000ffffu : 0u);
    }
    *reinterpret_cast<u32x4_t*>(vs + p * 16) = v;
  }
}

// max of a value with the value held by the lane 32 places away (the other half of the wave holds the
// other 16 keys of the same column): one v_permlane32_swap (swaps the upper half of its first operand
// with the lower half of its second; given the value twice, each result holds one half's values in
// both halves) instead of a round trip through the LDS crossbar
__device__ __forceinline__ float max_across_halves(float v) {
  const unsigned u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// One unit of 32 keys for the wave's 32 columns: scores, online softmax, P V.
// kst / vst: this lane's 16 bytes of the unit's first K fragment (step s at + s KB) and first V
// fragment ((db, u) at + (db * 2 + u) KB).  vis: visibility bits of this lane's 16 keys at bit
// 8 (v / 4) + v % 4 (register v <-> key 8 (v / 4) + 4 half + v % 4), used when `masked` (wave-uniform).
__device__ __forceinline__ void ring_unit(bool masked, const unsigned char* kst, const unsigned char* vst, unsigned vis, float scale,
                                          const bf16x8_t (&qf)[8], f32x16_t (&oacc)[4], float& m, float& l) {
  f32x16_t sc;
#pragma unroll
  for (int v = 0; v < 16; ++v) sc[v] = 0.f;
  // fragment reads run one step ahead of their MFMA and are pinned there (scheduling barriers): left
  // to itself the compiler hoists all of them and runs out of registers
  // the matrix phases run at raised wave priority: of the waves that share a SIMD, one with matrix
  // work issues first and the others fill the gaps with their softmax arithmetic
  // (the LDS answers after three to four MFMA times: PF reads are in flight, as many as the
  // registers allow)
  constexpr int PF = 3, NF = PF + 1;
  bf16x8_t fr[NF];
  // fragment j of the unit's 16: K steps 0..7, then V fragments in the order (u, db) = j - 8
  auto frag_at = [&](int j) {
    return j < 8 ? *reinterpret_cast<const bf16x8_t*>(kst + j * 1024)
                 : *reinterpret_cast<const bf16x8_t*>(vst + ((((j - 8) & 3) * 2) + ((j - 8) >> 2)) * 1024);
  };
#pragma unroll
  for (int j = 0; j < PF; ++j) fr[j] = frag_at(j);
  __builtin_amdgcn_s_setprio(2);
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    fr[(s + PF) % NF] = frag_at(s + PF);
    __builtin_amdgcn_sched_barrier(0);
    sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[s % NF], qf[s], sc, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
  __builtin_amdgcn_s_setprio(0);
  // scores stay unscaled; the scale is folded into the exponent: p = 2^(s*scale - m*scale)
  if (masked) {
#pragma unroll
    for (int v = 0; v < 16; ++v) sc[v] = ((vis >> (8 * (v >> 2) + (v & 3))) & 1u) ? sc[v] : NEG_BIG;
  }
  float tmax = fmaxf(sc[0], sc[1]);
#pragma unroll
  for (int v = 2; v < 16; v += 2) tmax = fmaxf(tmax, fmaxf(sc[v], sc[v + 1]));
  tmax = max_across_halves(tmax);
  const float m_new = tmax * scale > m * scale + RESCALE_SLACK ? tmax : m;
  // no key of the column visible so far (m_new at its start value): any finite reference does, the
  // masked scores' exponents then lie far below the range and their probabilities come out as 0
  const float mb = m_new > 0.5f * NEG_BIG ? m_new * scale : 0.f;
  // m still at its start value: nothing accumulated yet, nothing to scale
  const bool moved = m_new != m && m > 0.5f * NEG_BIG;
  if (__builtin_amdgcn_ballot_w64(moved) != 0ull) {
    const float alpha = m > 0.5f * NEG_BIG ? __builtin_amdgcn_exp2f(m * scale - mb) : 1.0f;
    l *= alpha;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) oacc[i][v] *= alpha;
  }
  m = m_new;
  __builtin_amdgcn_sched_barrier(0);
  // exponentials four at a time (fenced: all sixteen in flight at once cost registers the Q
  // fragments need), converted to the bf16 operand fragments as they come
  float lsum = 0.f;
  bf16x8_t pf[2];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int v = 4 * c + e;
      // a masked score is NEG_BIG: its exponent lies far below the range, p = 0 without a test
      float p = __builtin_amdgcn_exp2f(fmaf(sc[v], scale, -mb));
      lsum += p;
      pf[v >> 3][v & 7] = (bf16_t)p;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  l += lsum;
  __builtin_amdgcn_s_setprio(2);
  // O^T += V^T P^T: k-step u takes registers 8u..8u+7, i.e. keys 16u + {0, 8} + 4 half + 0..3 -- one
  // 16-byte read in the permuted LDS order
#pragma unroll
  for (int i = 0; i < 8; ++i) {                 // i = u * 4 + db
    const int u = i >> 2, db = i & 3;
    if (i + PF < 8) fr[(8 + i + PF) % NF] = frag_at(8 + i + PF);
    __builtin_amdgcn_sched_barrier(0);
    oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[(8 + i) % NF], pf[u], oacc[db], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
  __builtin_amdgcn_s_setprio(0);
}

// Waves of a workgroup with ct_wg column tiles and tps key tiles.  A wave has a whole column tile, or the even or odd
// half of each of its key tiles; the SIMD with the most half-tiles sets the pace (waves go to SIMDs round-robin).  Two
// waves share a column tile where that evens the SIMDs out: ct_wg = 9 gives loads of 5, 5, 4, 4 half-tiles instead of
// 6, 4, 4, 4; with one or two column tiles it puts idle SIMDs to work, where there are key tiles enough to make up for
// the exchange at the end (68 rows, 2048 keys, two column tiles: 20.1 -> 18.2 us; one key tile: 10.7 -> 11.3).  At least
// four waves (they carry the loads).
struct RingGeometry { int n_full, waves; };
__host__ __device__ inline RingGeometry ring_geometry(int ct_wg, int tps) {
  const int rem = ct_wg & 3;
  int paired = 0;
  if (ct_wg <= 2) paired = tps >= 3 ? ct_wg : 0;
  else if ((rem == 1 || rem == 2) && ct_wg > 4 && ct_wg + rem <= RING_MAX_WAVES) paired = rem;
  return {ct_wg - paired, ct_wg + paired < 4 ? 4 : ct_wg + paired};
}
// time of a key tile in a workgroup with that many column tiles, 10 ns
__host__ __device__ constexpr int ring_tile_time(int c) {
  constexpr int t[RING_MAX_WAVES] = {84, 70, 104, 110, 120, 126, 138, 150, 165, 175, 208, 218};
  return t[c - 1];
}
constexpr int PIECE_TIME = 180;                          // start and end of a workgroup's work on a sequence, 10 ns

// ---- batches: one line of work per kv head ----------------------------------------------------------------------
// The sequences of a batch differ in length and rows, which only the device knows.  A grid of equal splits of the longest
// one gives the CUs unequal work (16 sequences of 1638 to 8192 keys and 40 to 132 rows: a launch took 237 us, the longest
// sequence's single split 215 of them).  Instead the sequences' key tiles, each weighted with its time, form one line per kv
// head, which is cut into as many equal shares as there are workgroups; a share is one sequence's tiles, or the end of one,
// some whole ones and the start of another.  A column group of a share (q_tiles of them) is a workgroup of its own beside the others, so
// that they read the same keys at the same time.  Piece (sequence s, share w) leaves its partial in slot s + w, which
// rises along the line: pieces never share one, and those of a sequence are consecutive.
// Table of the cuts (ints): [0] shares; share w begins at tile [3 + 2 w] of sequence [2 + 2 w], w <= shares; then per sequence
// the first and the last share that has any of it.
constexpr int MAX_SHARES = 63, MAX_SHARED_SEQS = 2 * MAX_SHARES;
__host__ __device__ constexpr int cuts_of_seq(int max_shares) { return 2 + 2 * (max_shares + 1); }

// columns of a sequence in a workgroup: its column tiles spread evenly over the groups
__device__ __forceinline__ int even_ct(int ncols, int q_tiles) { return ((ncols + 31) / 32 + q_tiles - 1) / q_tiles; }

// One workgroup, a thread per sequence.  What is before a sequence on the line is a sum over the lanes; a thread that added up the
// sequences in front of its own, a chain of loads for each, took 8.4 us at 16 sequences and 29.9 at 126, this 4.6 and 3.7.
__global__ __launch_bounds__(128) void k_attn_cuts(BlockDev b, KvDev kv, int G, int q_tiles, int max_shares, int32_t* __restrict__ cuts) {
  static_assert(MAX_SHARED_SEQS <= 128, "a thread each");
  __shared__ int64_t first_wave, all;
  const int s = threadIdx.x;
  int w = 0, nt = 0, u = 1;                              // weight and key tiles of the sequence, and the weight of one
  if (s < b.batch) {
    const int nr = b.n_rows[s];
    if (seq_ok(kv, s, nr, b.rows_per_seq) && nr > 0) {
      nt = (kv.len[s] + nr + 63) >> 6;
      u = ring_tile_time(even_ct(nr * G, q_tiles));
      w = PIECE_TIME + nt * u;
    }
  }
  int64_t upto = w;                                      // of this sequence and those before it
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t x = __shfl_up(upto, o, 64);
    if ((s & 63) >= o) upto += x;
  }
  if (s == 63) first_wave = upto;
  __syncthreads();
  if (s >= 64) upto += first_wave;
  if (s == 127) all = upto;
  __syncthreads();
  const int64_t total = all, c0 = upto - w;
  // a share of less than about two key tiles costs more in its partial than it gives
  const int64_t shares = max((int64_t)1, min((int64_t)max_shares, total / 400));
  if (s == 0) {
    cuts[0] = (int)shares;
    cuts[2 + 2 * shares] = b.batch; cuts[3 + 2 * shares] = 0;
    if (total == 0) { cuts[2] = b.batch; cuts[3] = 0; }
  }
  if (s >= b.batch) return;
  int first = 0, last = -1;
  if (w > 0) {
    first = (int)min(shares - 1, c0 * shares / total);              // share x begins at x * total / shares
    while ((int64_t)first * total / shares > c0) --first;
    while (first + 1 < shares && (int64_t)(first + 1) * total / shares <= c0) ++first;
    last = first;
    while (last + 1 < shares && (int64_t)(last + 1) * total / shares < c0 + w) ++last;
    for (int x = first; x <= last; ++x) {
      const int64_t at = (int64_t)x * total / shares - c0;
      if (at < 0) continue;                                         // begins in a sequence before
      cuts[2 + 2 * x] = s;
      cuts[3 + 2 * x] = (int)min((int64_t)nt, max((int64_t)0, (at - PIECE_TIME + u - 1) / u));
    }
  }
  cuts[cuts_of_seq(max_shares) + 2 * s] = first;
  cuts[cuts_of_seq(max_shares) + 2 * s + 1] = last;
}

// the key tiles of sequence s, nt in all, that share w has
__device__ __forceinline__ void share_tiles(const int32_t* __restrict__ cuts, int w, int s, int nt, int& t0, int& t1) {
  t0 = cuts[2 + 2 * w] == s ? cuts[3 + 2 * w] : 0;
  t1 = cuts[4 + 2 * w] == s ? cuts[5 + 2 * w] : nt;
}

// LPW: 1 KB wave-loads per loading wave and tile (the first 32 / LPW waves of the workgroup load).  NT: K and V by
// nontemporal loads.
// CUTS: a share of a batch's line of work instead of one split of one sequence (cuts; nsplit: shares launched).
template <int LPW, bool PACKED, bool NT, bool CUTS>
__global__ __launch_bounds__(64 * RING_MAX_WAVES) void k_attn_ring(BlockDev b, KvDev kv, int layer, int hq, int hkv,
                                                                  const bf16_t* __restrict__ q,
                                                                  float* __restrict__ part_o,
                                                                  float* __restrict__ part_ml, int nsplit, int tps,
                                                                  int q_tiles, int ct_wg, int n_full_wg,
                                                                  const int32_t* __restrict__ cuts) {
  constexpr int HD = 128;
  extern __shared__ __align__(16) unsigned char lds[];
  hkv = with_args(hkv, b.n_rows, b.rows_per_seq, b.batch, b.anc, kv.len, kv.base, kv.seq_cap, kv.capacity);
  hkv = with_args(hkv, kv.len_bound, kv.k, kv.v, layer, hq, q, part_o, part_ml);
  hkv = with_args(hkv, nsplit, tps, q_tiles, ct_wg, n_full_wg, b.anc_words, cuts, part_ml);
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lg = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = hq / hkv;
  // XCD-aware logical id: the query tiles that stream the same keys (same kv head, same split) get
  // consecutive logical ids on one XCD and so share its L2; the shares of a kv head are neighbours too
  const int total_wg = CUTS ? q_tiles * hkv * nsplit : q_tiles * hkv * b.batch * nsplit;
  const int per_xcd = (total_wg + 7) >> 3;
  const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (logical >= total_wg) return;
  const int qt = logical % q_tiles;
  const int kvh = CUTS ? logical / (q_tiles * nsplit) : (logical / q_tiles) % hkv;
  const int zz = logical / (q_tiles * hkv);
  const int share = (logical / q_tiles) % nsplit;
  if (CUTS && share >= cuts[0]) return;
  const int seq_first = CUTS ? cuts[2 + 2 * share] : zz / nsplit;
  const int seq_last = CUTS ? min(cuts[4 + 2 * share], b.batch - 1) : seq_first;
  const int sp = zz % nsplit;

  auto piece = [&](int seq) {
  const int nr = b.n_rows[seq];
  if (!seq_ok<!CUTS>(kv, seq, nr, b.rows_per_seq)) return;
  const int ncols = nr * G;
  const int ct_own = CUTS ? even_ct(ncols, q_tiles) : ct_wg;   // column tiles of a workgroup
  if (qt * ct_own * 32 >= ncols) return;                // no live query column in this workgroup
  const int L = kv.len[seq], total = L + nr;
  const int ntiles = (total + 63) >> 6;
  int t0 = sp * tps, t1 = min(ntiles, t0 + tps);
  if (CUTS) share_tiles(cuts, share, seq, ntiles, t0, t1);
  const int nt = t1 - t0;
  if (CUTS && nt <= 0) return;
  // this wave's column tile inside the workgroup and the halves of every key tile it works on: waves
  // up to n_full take a whole tile each, the others pair up on one (first = keys 0..31 of a tile,
  // second = keys 32..63) and are merged at the end; waves beyond the tiles only help load
  int n_full = n_full_wg;
  if (CUTS) {
    const RingGeometry g = ring_geometry(ct_own, nt);
    n_full = g.waves * 64 <= (int)blockDim.x ? g.n_full : ct_own;
  }
  const int ctl = wave < n_full ? wave : n_full + ((wave - n_full) >> 1);
  const bool pair = wave >= n_full;
  const int kh_first = pair ? ((wave - n_full) & 1) : 0, kh_last = pair ? kh_first : 1;

  const int qcol = (qt * ct_own + ctl) * 32 + lr;
  const bool col_live = qcol < ncols;
  const bool wave_live = ctl < ct_own && (qt * ct_own + ctl) * 32 < ncols;  // wave-uniform
  const int r = col_live ? qcol / G : 0;
  const int h = kvh * G + (col_live ? qcol % G : 0);
  const size_t row = (size_t)seq * b.rows_per_seq + r;
  // partial of this wave's column tile and split: O^T as [feature][column] (a store instruction of
  // the wave covers whole 128-byte lines), then (m, l) per column
  const size_t n_ct = (size_t)q_tiles * ct_wg, ct = qt * ct_own + min(ctl, ct_own - 1);
  const size_t ptile = CUTS ? ((size_t)kvh * (b.batch + nsplit) + seq + share) * n_ct + ct
                            : (((size_t)seq * hkv + kvh) * n_ct + ct) * nsplit + sp;
  float* po = part_o + ptile * (HD * 32);
  float* pml = part_ml + ptile * 64;

  if (nt <= 0) {   // empty split: neutral partial
    if (wave_live && kh_first == 0) {
      for (int f = lg; f < HD; f += 2) po[f * 32 + lr] = 0.f;
      if (lg == 0) { pml[lr * 2] = NEG_BIG; pml[lr * 2 + 1] = 0.f; }
    }
    return;
  }

  // ---- ring: tile i of the split lives in stage i % 4; piece p of a tile (1 KB) is K piece p for
  // p < 16, V piece p - 16 otherwise; loading wave w brings pieces w * LPW .. w * LPW + LPW - 1
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  const bool loader = wave < 32 / LPW;
  const int64_t base = kv.base[seq];
  const unsigned char* kt0 =
      reinterpret_cast<const unsigned char*>((const bf16_t*)kv.k + kv_plane(layer, kvh, hkv, kv.capacity, HD) + (size_t)base * HD);
  const unsigned char* vt0 =
      reinterpret_cast<const unsigned char*>((const bf16_t*)kv.v + kv_plane(layer, kvh, hkv, kv.capacity, HD) + (size_t)base * HD);
  const int piece0 = wave * LPW;                        // wave-uniform
  const unsigned char* src0 = (piece0 < 16 ? kt0 : vt0) + (size_t)(piece0 & 15) * 1024;
  const uint32_t lane_off = (uint32_t)lane * 16;
  auto issue_tile = [&](int i) {
    if (!loader) return;
    const unsigned char* src = src0 + (size_t)(t0 + i) * K_TILE_BYTES;
    const uint32_t dst = lds0 + (i & 3) * STAGE_BYTES + piece0 * 1024;
    load_to_lds16_sbase<0, NT>(src, lane_off, dst);
    load_to_lds16_sbase<1024, NT>(src, lane_off, dst);
    load_to_lds16_sbase<2048, NT>(src, lane_off, dst);
    load_to_lds16_sbase<3072, NT>(src, lane_off, dst);
    if (LPW == 8) {
      load_to_lds16_sbase<0, NT>(src + 4096, lane_off, dst + 4096);
      load_to_lds16_sbase<1024, NT>(src + 4096, lane_off, dst + 4096);
      load_to_lds16_sbase<2048, NT>(src + 4096, lane_off, dst + 4096);
      load_to_lds16_sbase<3072, NT>(src + 4096, lane_off, dst + 4096);
    }
  };
  // Q^T fragments: lane = query column, 8 features per k-step at 16 s + 8 lg.  The compiler places
  // waits on the load counter for the loads it knows of, and one of those inside the tile loop would
  // also drain the ring's prefetches (which it does not know of).  So the fragments are loaded
  // between the first tile's loads and the others', and an empty statement that names them right
  // after makes the compiler wait for them here: by then the first tile (older, loads retire in
  // order) has landed too, which the first iteration needs anyway, and no load of the compiler's is
  // left in flight when the loop starts.
  issue_tile(0);
  bf16x8_t qf[8];
  {
    const bf16_t* qp = q + (act_row<PACKED>(b, seq, r) * hq + h) * HD + 8 * lg;
#pragma unroll
    for (int s = 0; s < 8; ++s) qf[s] = *reinterpret_cast<const bf16x8_t*>(qp + 16 * s);
    asm volatile("" : "+v"(qf[0]), "+v"(qf[1]), "+v"(qf[2]), "+v"(qf[3]), "+v"(qf[4]), "+v"(qf[5]), "+v"(qf[6]), "+v"(qf[7])
                 :: "memory");
  }
  if (nt > 1) issue_tile(1);
  if (nt > 2) issue_tile(2);
  const uint64_t* anc = b.anc + row * b.anc_words;
  const float scale = LOG2E / sqrtf((float)HD);
  f32x16_t oacc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[i][v] = 0.f;
  float m = NEG_BIG, l = 0.f;

  const unsigned char* frag = lds + lane * 16;          // this lane's 16 bytes of fragment 0 of stage 0
  for (int i = 0; i < nt; ++i) {
    // tile i has landed (this wave's loads: they retire in order and the tiles after i stay in
    // flight; the barrier covers the other waves'); every wave is done with tile i - 1, whose stage
    // takes tile i + 3
    if (i + 2 < nt) wait_loads_but<2 * LPW>();
    else if (i + 1 < nt) wait_loads_but<LPW>();
    else wait_loads_but<0>();
    __syncthreads();
    if (i + 3 < nt) issue_tile(i + 3);
    const int key0 = (t0 + i) * 64;
    const int keys_left = total - key0;
    if (keys_left < 64) {
      ring_zero_tail(lds + (i & 3) * STAGE_BYTES + K_TILE_BYTES, keys_left, tid, blockDim.x);
      __syncthreads();
    }
    if (!wave_live) continue;
    const unsigned char* st = frag + (i & 3) * STAGE_BYTES;
    const bool masked = key0 + 64 > L;                   // the tile touches the block rows or the sequence's end
    uint64_t wnd = 0;
    if (masked) wnd = key_window(anc, b.anc_words, key0 - L, keys_left);
    if (kh_first == 0) ring_unit(masked, st, st + K_TILE_BYTES, (unsigned)wnd >> (4 * lg), scale, qf, oacc, m, l);
    if (kh_last == 1)
      ring_unit(masked, st + 8192, st + K_TILE_BYTES + 8192, (unsigned)(wnd >> 32) >> (4 * lg), scale, qf, oacc, m, l);
  }

  l += __shfl_xor(l, 32, 64);
  if (n_full < ct_own) {
    // paired waves: the second hands its (m, l, O) to the first through LDS (the ring is free now)
    __syncthreads();
    float* xo = reinterpret_cast<float*>(lds) + (size_t)(ctl - n_full) * (HD * 32 + 64);
    if (pair && kh_first == 1 && wave_live) {
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) xo[(db * 16 + v) * 64 + lane] = oacc[db][v];
      if (lg == 0) { xo[HD * 32 + lr * 2] = m; xo[HD * 32 + lr * 2 + 1] = l; }
    }
    __syncthreads();
    if (pair && kh_first == 0 && wave_live) {
      const float mo = xo[HD * 32 + lr * 2], lo = xo[HD * 32 + lr * 2 + 1];
      const float mm = fmaxf(m, mo);
      // a side that saw no visible key (m at its start value) holds nothing: weight it out
      const float wa = m > 0.5f * NEG_BIG ? __builtin_amdgcn_exp2f((m - mm) * scale) : 0.f;
      const float wb = mo > 0.5f * NEG_BIG ? __builtin_amdgcn_exp2f((mo - mm) * scale) : 0.f;
      l = l * wa + lo * wb;
      m = mm;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[db][v] = oacc[db][v] * wa + xo[(db * 16 + v) * 64 + lane] * wb;
    }
  }
  if (wave_live && kh_first == 0) {
    // register v of feature block db <-> feature db*32 + 8*(v/4) + 4*lg + v%4
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) po[(db * 32 + 8 * (v >> 2) + 4 * lg + (v & 3)) * 32 + lr] = oacc[db][v];
    if (lg == 0) { pml[lr * 2] = m * scale; pml[lr * 2 + 1] = l; }   // m in the exponent's units
  }
  };
  for (int seq = seq_first; seq <= seq_last; ++seq) {
    if (CUTS && seq > seq_first) {                      // the last piece's stores do not count as loads of this one; everyone is done with the LDS
      wait_loads_but<0>();
      __syncthreads();
    }
    piece(seq);
  }
}

// --------------------------------------------------------------------------------------------------
__device__ __forceinline__ void store4(float* dst, f32x4_t v) { *reinterpret_cast<f32x4_t*>(dst) = v; }
__device__ __forceinline__ void store4(bf16_t* dst, f32x4_t v) {
  bf16x4_t o = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
  *reinterpret_cast<bf16x4_t*>(dst) = o;
}

// Merge of the per-split partials, in split order.  hd/4 threads per (row, head) item, four
// features each; a 256-thread workgroup takes 256/(hd/4) items.
template <typename T, bool PACKED>
__global__ __launch_bounds__(256) void k_attn_merge(BlockDev b, KvDev kv, int hq, int hd,
                                                    const float* __restrict__ part_o,
                                                    const float* __restrict__ part_ml, int nsplit,
                                                    T* __restrict__ out, int n_items) {
  const int per = hd >> 2;
  const int item = blockIdx.x * (256 / per) + threadIdx.x / per;   // row * hq + h
  const int d = (threadIdx.x % per) * 4;
  if (item >= n_items) return;
  const int row = item / hq;
  const int seq = row / b.rows_per_seq, r = row % b.rows_per_seq;
  const int nr = b.n_rows[seq];
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  if (!seq_ok(kv, seq, nr, b.rows_per_seq) || r >= nr) {
    if (!PACKED) store4(out + (size_t)item * hd + d, acc);
    return;
  }
  T* dst = out + (act_row<PACKED>(b, seq, r) * hq + item % hq) * hd + d;
  const size_t item0 = (size_t)item * nsplit;
  float mx = NEG_BIG;
  for (int s = 0; s < nsplit; ++s) mx = fmaxf(mx, part_ml[(item0 + s) * 2]);
  float lt = 0.f;
  for (int s = 0; s < nsplit; ++s) {
    const float w = exp2f(part_ml[(item0 + s) * 2] - mx);
    lt += part_ml[(item0 + s) * 2 + 1] * w;
    const f32x4_t o = *reinterpret_cast<const f32x4_t*>(part_o + (item0 + s) * hd + d);
    acc += o * w;
  }
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  store4(dst, acc * inv);
}

// Merge for the ring kernel's partial layout ([column tile][split][feature][column]), in split
// order.  A workgroup of 256 threads takes 32 features of one column tile of 32 query columns.
// First the weights 2^(m_s - max) of the tile's columns and splits: thread (split group, column)
// fetches the (m, l) of every eighth split at once -- one after the other, a column's splits would
// cost a memory latency each -- and the eight groups combine through LDS.  Then thread (column,
// feature quad) sums the splits' O, every load instruction of a wave covering whole 128-byte lines.
// CUTS: the pieces of a sequence in the shares of its batch's line (nsplit: shares launched).
template <int MAXS, bool PACKED, bool CUTS>
__global__ __launch_bounds__(256) void k_attn_merge_ring(BlockDev b, KvDev kv, int hq, int hkv,
                                                         const float* __restrict__ part_o,
                                                         const float* __restrict__ part_ml, int nsplit,
                                                         int n_ct, bf16_t* __restrict__ out, const int32_t* __restrict__ cuts) {
  constexpr int HD = 128, PER = MAXS / 8;
  __shared__ int slots[CUTS ? MAXS : 1], n_slots[1];
  __shared__ float w_s[MAXS][32];
  __shared__ float red[8][32];
  __shared__ float red_l[8][32];
  n_ct = with_args(n_ct, b.n_rows, b.rows_per_seq, kv.len, kv.base, kv.seq_cap, kv.capacity, kv.len_bound, b.batch);
  n_ct = with_args(n_ct, hq, hkv, part_o, part_ml, nsplit, out, cuts, hq);
  const int G = hq / hkv;
  const int fq = blockIdx.x & 3;
  const int tile = blockIdx.x >> 2;                 // (seq * hkv + kvh) * n_ct + ct
  const int ct = tile % n_ct, kvh = (tile / n_ct) % hkv, seq = tile / (n_ct * hkv);
  const int nr = b.n_rows[seq];
  const bool ok = seq_ok<true>(kv, seq, nr, b.rows_per_seq);
  const int col = threadIdx.x & 31, grp = threadIdx.x >> 5;
  const int c = ct * 32 + col;                      // column within the kv group
  const bool live = ok && c < nr * G;
  const bool in_block = PACKED ? live : c < b.rows_per_seq * G;     // has an output row at all
  size_t t0 = (size_t)tile * nsplit, step = 1;          // first partial of the column tile, and how far apart they are
  if constexpr (CUTS) {
    const int32_t* ends = cuts + cuts_of_seq(nsplit) + 2 * seq;
    const int first = ends[0], pieces = ok ? ends[1] - first + 1 : 0;   // at most 63
    if (threadIdx.x < 64) {
      int a = 0, e = 0;
      if ((int)threadIdx.x < pieces) share_tiles(cuts, first + threadIdx.x, seq, (kv.len[seq] + nr + 63) >> 6, a, e);
      const uint64_t there = __builtin_amdgcn_ballot_w64(a < e);
      if (a < e) slots[__popcll(there & ((1ull << threadIdx.x) - 1ull))] = seq + first + threadIdx.x;
      if (threadIdx.x == 0) n_slots[0] = __popcll(there);
    }
    __syncthreads();
    t0 = (size_t)kvh * (b.batch + nsplit) * n_ct + ct;
    step = n_ct;
    nsplit = n_slots[0];
  }
  auto part = [&](int sp) { return t0 + (CUTS ? (size_t)slots[sp] : (size_t)sp) * step; };
  // O of the first splits is on its way before their weights are known: one memory latency instead of two, 68 rows on 2048 keys
  // 5.3 -> 4.7 us (sixteen of them no better)
  constexpr int EARLY = 8;
  const int f0 = fq * 32 + grp * 4;
  const float* p = part_o + (size_t)f0 * 32 + col;
  float early[EARLY][4];
#pragma unroll
  for (int s = 0; s < EARLY; ++s)
    if (s < nsplit) {
#pragma unroll
      for (int e = 0; e < 4; ++e) early[s][e] = p[part(s) * (HD * 32) + 32 * e];
    }
  float ms[PER], ls[PER];
  float mx = NEG_BIG;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int sp = grp + 8 * i;
    ms[i] = NEG_BIG; ls[i] = 0.f;
    if (live && sp < nsplit) {
      const float2 ml = *reinterpret_cast<const float2*>(part_ml + part(sp) * 64 + col * 2);
      ms[i] = ml.x; ls[i] = ml.y;
    }
    mx = fmaxf(mx, ms[i]);
  }
  red[grp][col] = mx;
  __syncthreads();
#pragma unroll
  for (int g = 0; g < 8; ++g) mx = fmaxf(mx, red[g][col]);
  float lt = 0.f;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int sp = grp + 8 * i;
    const float w = exp2f(ms[i] - mx);
    if (sp < nsplit) w_s[sp][col] = w;
    lt += ls[i] * w;
  }
  red_l[grp][col] = lt;
  __syncthreads();
  if (!in_block) return;
  // the splits' sums are added in group order: fixed, like everything else here
  lt = 0.f;
#pragma unroll
  for (int g = 0; g < 8; ++g) lt += red_l[g][col];
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  if (live) {
#pragma unroll
    for (int s = 0; s < EARLY; ++s)
      if (s < nsplit) {
        const float w = w_s[s][col];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += early[s][e] * w;
      }
#pragma unroll 8
    for (int s = EARLY; s < nsplit; ++s) {
      const float w = w_s[s][col];
      const float* ps = p + part(s) * (HD * 32);
      acc[0] += ps[0] * w; acc[1] += ps[32] * w; acc[2] += ps[64] * w; acc[3] += ps[96] * w;
    }
    acc *= inv;
  }
  const int r = c / G, h = kvh * G + c % G;
  store4(out + (act_row<PACKED>(b, seq, r) * hq + h) * HD + f0, acc);
}

}  // namespace

// the ring kernel uses more dynamic LDS than a kernel gets by default: raise the limit once (also
// called when a context is created, so that no launch inside a stream capture is the first one)
hipError_t attn_prepare() {
  static const hipError_t attr = [] {
    for (const void* k : {reinterpret_cast<const void*>(k_attn_ring<4, false, false, false>), reinterpret_cast<const void*>(k_attn_ring<4, false, false, true>),
                          reinterpret_cast<const void*>(k_attn_ring<4, false, true, false>), reinterpret_cast<const void*>(k_attn_ring<4, false, true, true>),
                          reinterpret_cast<const void*>(k_attn_ring<4, true, false, false>), reinterpret_cast<const void*>(k_attn_ring<4, true, false, true>),
                          reinterpret_cast<const void*>(k_attn_ring<4, true, true, false>), reinterpret_cast<const void*>(k_attn_ring<4, true, true, true>),
                          reinterpret_cast<const void*>(k_attn_ring<8, false, false, false>), reinterpret_cast<const void*>(k_attn_ring<8, false, false, true>),
                          reinterpret_cast<const void*>(k_attn_ring<8, false, true, false>), reinterpret_cast<const void*>(k_attn_ring<8, false, true, true>),
                          reinterpret_cast<const void*>(k_attn_ring<8, true, false, false>), reinterpret_cast<const void*>(k_attn_ring<8, true, false, true>),
                          reinterpret_cast<const void*>(k_attn_ring<8, true, true, false>), reinterpret_cast<const void*>(k_attn_ring<8, true, true, true>)}) {
      const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, RING_LDS_BYTES);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }();
  return attr;
}

namespace {
// most partial column tiles (column tiles x splits) of a plan, per sequence and kv head: what the workspace holds
int ring_tiles_bound(int cols) {
  const int ct = (cols + 31) / 32, q = (ct + RING_MAX_WAVES - 1) / RING_MAX_WAVES;
  return q * ((ct + q - 1) / q) * 64;
}

// Splits of the key range alone: rounds over the CUs x (tiles + about four tiles' time of a workgroup's own).
void plan_splits(AttnPlan& p, int base, int nt) {
  int best = 1, best_cost = 1 << 30;
  for (int ns = 1; ns <= 64; ++ns) {
    const int tps = (nt + ns - 1) / ns;
    if (ns > 1 && tps < 2) break;
    if ((nt + tps - 1) / tps != ns) continue;             // same partition as a smaller count
    const int cost = (base * ns + 255) / 256 * (tps + 4);
    if (cost < best_cost) { best_cost = cost; best = ns; }
  }
  p.tiles_per_split = (nt + best - 1) / best;
  p.nsplit = (nt + p.tiles_per_split - 1) / p.tiles_per_split;
}
}  // namespace

AttnPlan attn_plan(int dtype, int hd, int batch, int rows_per_seq, int hq, int hkv, int len_bound) {
  AttnPlan p;
  const int nt = (len_bound + rows_per_seq + 63) / 64;
  const int cols = rows_per_seq * (hq / hkv), ct = (cols + 31) / 32;
  if (dtype != ESP_BF16 || hd != 128) {
    // generic kernel: one wave per (row, head, split), as long as that is no more than 16 waves a CU.  A split more is a
    // serial step more of the merge, a split fewer a longer chain of key tiles: about twice the square root of their number
    // (one fp32 row, 4000 keys: 27.7 us in 63 splits, 16.4 in 16, 19.9 in 8; 16000 keys: 34.7, 36.1, and 29.8 in 32)
    const int64_t waves = (int64_t)batch * rows_per_seq * hq;
    int most = 1;
    while (most < 64 && most < nt && (int64_t)most * most < 4 * (int64_t)nt) ++most;
    const int ns = (int)std::max<int64_t>(1, std::min<int64_t>(most, 4096 / waves));
    p.tiles_per_split = (nt + ns - 1) / ns;
    p.nsplit = (nt + p.tiles_per_split - 1) / p.tiles_per_split;
    return p;
  }
  p.q_tiles = (ct + RING_MAX_WAVES - 1) / RING_MAX_WAVES;
  p.ct_wg = (ct + p.q_tiles - 1) / p.q_tiles;
  plan_splits(p, p.q_tiles * hkv * batch, nt);
  // Column tiles per workgroup (one workgroup per CU) and splits of the key range together.  More column tiles share
  // each key tile's loads; more splits fill the CUs, but every one costs a partial (m, l, O) per column tile (16 KB,
  // written and read back).  Cost of a candidate in units of 10 ns: the two launches + rounds over the CUs x (start and
  // end of a workgroup + its key tiles x the time of one: the SIMD with the most half-tiles, or the loads of 32 KB with
  // that many CUs at it) + merge per partial column tile.  Fitted to 7200 measured candidates of 240 shapes (1 to 512 rows,
  // 64 to 32768 keys, batches of 1 to 16; model within 7 %).  The plan above (as many column tiles as twelve waves hold)
  // stays unless the model sees 4 % in another.  Where the model was too hopeful, against measured times of 469 shapes with the
  // cache out of the last-level cache: one or two column tiles take longer with all CUs at it; and a single split with four or
  // more column tiles, which leaves all masked key tiles of a column to one wave, was 3 to 11 % slower than the plan above where
  // that is one round too (five sequences of 200 rows on 600 keys 38.6 us, 35.1 in two splits; three of 320 on 256 keys 35.4, 30.3), and
  // with nearly every CU on one long split 25 us of 260 (eight sequences of 200 rows on 8192 keys, in a step).  Over the
  // shapes 0.948 of the plan above's time on average, four of them slower by 2 to 4.5 %, the others by at most 1.5 %.
  // Attention and merge of a layer: 90 rows on 2048 keys 26.6 -> 19.6 us, 132 rows on 1000 keys 24.5 -> 17.6.
  auto cost = [&](int q, int c, int ns, int tps) {
    const int64_t groups = (int64_t)q * hkv * batch, rounds = (groups * ns + 255) / 256, busy = std::min<int64_t>(groups * ns, 256);
    const bool short_unpaired = c <= 2 && tps < 3;
    const int64_t tile = std::max<int64_t>(short_unpaired ? 104 : ring_tile_time(c) + (c <= 2 ? 6 * busy / 256 : 0), 80 * busy / 256);
    return 880 + rounds * ((short_unpaired ? 160 : 180) + tps * tile) + groups * c * ns * 55 / 100;
  };
  const int64_t base_wg = (int64_t)p.q_tiles * hkv * batch * p.nsplit;
  const bool base_split = p.nsplit > 1;
  int64_t best_cost = cost(p.q_tiles, p.ct_wg, p.nsplit, p.tiles_per_split) * 96 / 100;
  for (int want = std::min(ct, RING_MAX_WAVES); want >= 1; --want) {
    const int q = (ct + want - 1) / want, c = (ct + q - 1) / q;
    if (c != want) continue;                              // the same tiling as with fewer
    const int most = std::min(64, ring_tiles_bound(cols) / (q * c));
    for (int ns = 1; ns <= most && ns <= nt; ++ns) {
      const int tps = (nt + ns - 1) / ns;
      if (ns > 1 && tps < 2) break;                       // (one row, 400 keys: 10.6 us in four splits, 11.1 in seven)
      if ((nt + tps - 1) / tps != ns) continue;           // same partition as a smaller count
      int64_t t = cost(q, c, ns, tps);
      if (ns == 1 && c >= 4 && base_split) {
        if (base_wg <= 256 && tps >= 5) continue;
        if (tps > 64 && (int64_t)q * hkv * batch > 240) t = t * 103 / 100;
      }
      if (t < best_cost) {
        best_cost = t;
        p.nsplit = ns; p.tiles_per_split = tps; p.q_tiles = q; p.ct_wg = c;
      }
      if ((int64_t)q * hkv * batch * ns > 16 * 256) break;   // more splits even out nothing any more
    }
  }
  return p;
}

size_t attn_partial_floats_bound(int dtype, int batch, int rows_per_seq, int hq, int hkv, int hd) {
  if (dtype == ESP_BF16 && hd == 128)   // ring layout: whole column tiles of 32
    return (size_t)batch * hkv * ring_tiles_bound(rows_per_seq * (hq / hkv)) * (32 * (hd + 2));
  return (size_t)batch * rows_per_seq * hq * 64 * (hd + 2);
}

// The generic kernel merges its splits itself where they are waves that a workgroup can hold with the registers they take.
constexpr int GENERIC_WAVES_64 = 8, GENERIC_WAVES_128 = 4;
// And only where all workgroups have a place at once: their waves share a CU four at a time or more, a workgroup waits for room for all of
// its own and none leaves before the last (200 rows of four heads on 4000 keys, five splits: 73 us in two launches, 121 in one; four
// sequences of 60 rows on 1000 keys, HD 128, three splits: 76 and 92).  A single split merges nothing and always does.
bool attn_generic_merges(int hd, const AttnPlan& p, int64_t groups) {
  const int room = hd == 64 ? 12 : 4;                    // waves of a CU
  return p.nsplit <= (hd == 64 ? GENERIC_WAVES_64 : GENERIC_WAVES_128) && (p.nsplit == 1 || groups <= 256 * (p.nsplit > 4 ? 1 : room / p.nsplit));
}

// Shares of a batch's line of work per kv head: as many as there are CUs for them; 0: a grid of equal splits.  The line costs up to 3 us a
// layer (the cuts are looked up, a workgroup's second piece starts cold, more partials) and one launch a forward pass, so only
// where the longest sequence's split takes 45 us or more.  Steps of the 8B shape, a grid and shares, sequences of equal length and of an
// eighth to all of it: four layers, 16 of 132 rows on 16384 keys 5.54 -> 5.53 and 4.99 -> 4.60 ms, 8 of 68 on 8192 1416 -> 1429 and 1351
// -> 1331 us, 6 of 132 on 4096 1699 -> 1705 and 1632 -> 1591; 32 layers, 16 of 132 on 2048 28.4 -> 28.75 and 28.14 -> 28.17 ms, 3 of
// 132 on 16384 11.45 -> 11.60.  Below the line: 6 of 200 rows, 2048 keys, attention of a layer 72 -> 73 and 66 -> 63 us (106 to 200
// rows of one length 66 -> 74); eight layers, 16 sequences of one row on 128 keys 816 -> 866.
// And only where the shares, 63 a kv head at most, have work for three quarters of the CUs, with two sequences to a share at most: one
// or two kv heads had 63 or 126 workgroups (256 sequences of one row, 4000 keys, one kv head 87 -> 290 us; 64 on 8000 keys, two kv heads
// 89 -> 142), and a grid of several rounds evens itself out (128 sequences of one row on 4096 keys, four layers 1990 -> 2060 us, 1535 ->
// 1555 with lengths of an eighth to all; 64 of them 1202 -> 1165 and 945 -> 905).
int attn_shares(int dtype, int hd, int batch, int rows_per_seq, int hq, int hkv, const AttnPlan& p) {
  if (dtype != ESP_BF16 || hd != 128 || batch < 2 || p.tiles_per_split * ring_tile_time(p.ct_wg) < 4500) return 0;
  // (batch + shares) x column tiles are what a share of the reserved partials holds
  const int room = batch * (ring_tiles_bound(rows_per_seq * (hq / hkv)) / (p.q_tiles * p.ct_wg) - 1);
  const int n = std::min(std::min(256 / (hkv * p.q_tiles), MAX_SHARES), room);
  return n < 2 || n * hkv * p.q_tiles < 192 || batch > 2 * n ? 0 : n;
}
size_t attn_cuts_ints(int batch) { return cuts_of_seq(MAX_SHARES) + 2 * (size_t)batch; }

hipError_t launch_attn_cuts(hipStream_t st, const BlockDev& b, const KvDev& kv, int hq, int hkv, const AttnPlan& p, int shares, int32_t* cuts) {
  if (b.batch > MAX_SHARED_SEQS) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_attn_cuts, dim3(1), dim3(128), 0, st, b, kv, hq / hkv, p.q_tiles, shares, cuts);
  return hipGetLastError();
}

size_t attn_partial_floats(int dtype, int batch, int rows_per_seq, int hq, int hkv, int hd, const AttnPlan& p) {
  if (dtype == ESP_BF16 && hd == 128) {
    const size_t whole = (size_t)p.q_tiles * p.ct_wg * hkv * (32 * (hd + 2)), shares = attn_shares(dtype, hd, batch, rows_per_seq, hq, hkv, p);
    return whole * std::max((size_t)batch * p.nsplit, shares ? batch + shares : 0);
  }
  return (size_t)batch * rows_per_seq * hq * p.nsplit * (hd + 2);
}

hipError_t launch_attn(hipStream_t st, int dtype, const BlockDev& b, const KvDev& kv, int layer, int hq, int hkv,
                       int hd, const void* q, float* partials, const AttnPlan& p, const int32_t* cuts, void* out) {
  const int M = b.batch * b.rows_per_seq;
  const bool packed = b.packed != nullptr;
  float* part_o = partials;
  float* part_ml = partials + (size_t)M * hq * p.nsplit * hd;
  if (dtype == ESP_BF16 && hd == 128) {
    const int shares = cuts ? attn_shares(dtype, hd, b.batch, b.rows_per_seq, hq, hkv, p) : 0, nsplit = shares ? shares : p.nsplit;
    const RingGeometry g = ring_geometry(p.ct_wg, shares ? 64 : p.tiles_per_split);
    part_ml = partials + (size_t)hkv * p.q_tiles * p.ct_wg * (shares ? b.batch + shares : b.batch * p.nsplit) * (32 * hd);
    const int total_wg = p.q_tiles * hkv * (shares ? shares : b.batch * p.nsplit);
    const hipError_t attr = attn_prepare();
    if (attr != hipSuccess) return attr;
    const dim3 grid(((total_wg + 7) / 8) * 8), block(64 * g.waves);
    // Nontemporal where a key tile is read by one workgroup only.  Eight layers of the 8B shape, this alone: one row on 32768 keys
    // 994 -> 952 us, 68 rows 1357 -> 1341, 16 sequences of one row on 8192 keys 1717 -> 1626; up to 2048 keys within 1 %.  Where
    // several workgroups read a tile, 50 and 80 rows got 1 % slower with it and the others stayed the same.
    const auto pick = [&](auto nt, auto line) {
      constexpr bool NT = decltype(nt)::value, CUTS = decltype(line)::value;
      return g.waves >= 8 ? (packed ? k_attn_ring<4, true, NT, CUTS> : k_attn_ring<4, false, NT, CUTS>)
                          : (packed ? k_attn_ring<8, true, NT, CUTS> : k_attn_ring<8, false, NT, CUTS>);
    };
    const std::true_type yes;
    const std::false_type no;
    const auto kern = shares ? (p.q_tiles == 1 ? pick(yes, yes) : pick(no, yes)) : (p.q_tiles == 1 ? pick(yes, no) : pick(no, no));
    hipLaunchKernelGGL(kern, grid, block, RING_LDS_BYTES, st, b, kv, layer, hq, hkv, (const bf16_t*)q, part_o, part_ml, nsplit,
                       p.tiles_per_split, p.q_tiles, p.ct_wg, g.n_full, cuts);
  } else {
    const bool vec = (((uintptr_t)kv.k | (uintptr_t)kv.v) & 15) == 0, merge = attn_generic_merges(hd, p, (int64_t)M * hq);
    const dim3 grid(M, hq, merge ? 1 : p.nsplit), block(merge ? 64 * p.nsplit : 64);
#define ESP_GENERIC(T_, HD_, P_)                                                                                             \
  do {                                                                                                                       \
    constexpr int W = HD_ == 64 ? GENERIC_WAVES_64 : GENERIC_WAVES_128;                                                      \
    const auto kern = merge ? (vec ? k_attn_generic<T_, HD_, P_, true, W> : k_attn_generic<T_, HD_, P_, false, W>)           \
                            : (vec ? k_attn_generic<T_, HD_, P_, true, 0> : k_attn_generic<T_, HD_, P_, false, 0>);          \
    hipLaunchKernelGGL(kern, grid, block, 0, st, b, kv, layer, hq, hkv, (const T_*)q, part_o, part_ml, p.nsplit,             \
                       p.tiles_per_split, (T_*)out);                                                                         \
  } while (0)
    if (dtype == ESP_F32 && hd == 64) ESP_GENERIC(float, 64, false);   // fp32 batches are not packed
    else if (dtype == ESP_F32 && hd == 128) ESP_GENERIC(float, 128, false);
    else if (dtype == ESP_BF16 && hd == 64 && packed) ESP_GENERIC(bf16_t, 64, true);
    else if (dtype == ESP_BF16 && hd == 64) ESP_GENERIC(bf16_t, 64, false);
#undef ESP_GENERIC
    else
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_attn_merge(hipStream_t st, int dtype, const BlockDev& b, const KvDev& kv, int hq, int hkv, int hd,
                             const float* partials, const AttnPlan& p, void* out, const int32_t* cuts) {
  const bool packed = b.packed != nullptr;
  if (dtype == ESP_BF16 && hd == 128) {
    const int n_ct = p.q_tiles * p.ct_wg;
    const float* part_o = partials;
    const int shares = cuts ? attn_shares(dtype, hd, b.batch, b.rows_per_seq, hq, hkv, p) : 0;
    const float* part_ml = partials + (size_t)hkv * n_ct * (shares ? b.batch + shares : b.batch * p.nsplit) * (32 * hd);
    const dim3 grid(b.batch * hkv * n_ct * 4);
    if (p.nsplit > 64) return hipErrorInvalidValue;
    const auto kern = shares ? (packed ? k_attn_merge_ring<64, true, true> : k_attn_merge_ring<64, false, true>)
                             : (packed ? k_attn_merge_ring<64, true, false> : k_attn_merge_ring<64, false, false>);
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, b, kv, hq, hkv, part_o, part_ml, shares ? shares : p.nsplit, n_ct, (bf16_t*)out, cuts);
    return hipGetLastError();
  }
  const int M = b.batch * b.rows_per_seq;
  if (attn_generic_merges(hd, p, (int64_t)M * hq)) return hipSuccess;   // done by the attention launch
  const float* part_o = partials;
  const float* part_ml = partials + (size_t)M * hq * p.nsplit * hd;
  const int n_items = M * hq, per_wg = 256 / (hd / 4);
  const dim3 grid((n_items + per_wg - 1) / per_wg);
  if (dtype == ESP_F32)
    hipLaunchKernelGGL((k_attn_merge<float, false>), grid, dim3(256), 0, st, b, kv, hq, hd, part_o, part_ml, p.nsplit,
                       (float*)out, n_items);
  else
    hipLaunchKernelGGL((packed ? k_attn_merge<bf16_t, true> : k_attn_merge<bf16_t, false>), grid, dim3(256), 0, st, b, kv, hq, hd, part_o, part_ml, p.nsplit,
                       (bf16_t*)out, n_items);
  return hipGetLastError();
}
