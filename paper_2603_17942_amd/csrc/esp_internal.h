// Internal declarations shared by the HIP sources of libesp_hip.so (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <vector>

#include "esp.h"

typedef __bf16 bf16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));   // 16 raw bytes in registers

#define ESP_WAVE 64

// ---- element conversion -----------------------------------------------------------------
__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return (bf16_t)v; }  // RNE

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// ---- direct global -> LDS loads --------------------------------------------------------------
// One 16-byte piece per lane from global memory straight into LDS (no register hop): a wave-uniform base address (scalar
// registers) plus a per-lane byte offset, the wave's 64 pieces land at lds_addr + 16 * lane.  The constant offset IMM is added to
// the global address and to the LDS address alike (piece j of a run: IMM = j KB, lds_addr the address of piece 0), so one vector
// register serves any number of pieces.  Issued as text so that the compiler's wait-count bookkeeping knows nothing of it: the
// LDS rings of the GEMM and attention kernels count their own loads (they retire in order) and would otherwise be
// drained before every LDS read.
// M0 (the LDS base of the transfer) is put back to what it held before, so the statement leaves no
// register changed that the compiler might rely on.  NT: nontemporal, for data that one workgroup (or a few at the same time)
// reads once.
template <int IMM, bool NT = false>
__device__ __forceinline__ void load_to_lds16_sbase(const void* sbase, uint32_t lane_off, uint32_t lds_addr) {
  uint32_t keep;
  if constexpr (NT)
    asm volatile(
        "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3 offset:%4 nt\n\ts_mov_b32 m0, %0"
        : "=&s"(keep)
        : "s"(lds_addr), "v"(lane_off), "s"(sbase), "n"(IMM)
        : "memory");
  else
    asm volatile(
        "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3 offset:%4\n\ts_mov_b32 m0, %0"
        : "=&s"(keep)
        : "s"(lds_addr), "v"(lane_off), "s"(sbase), "n"(IMM)
        : "memory");
}
template <int N_YOUNGER>
__device__ __forceinline__ void wait_loads_but() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N_YOUNGER) : "memory");
}

// ---- sample matching (temperature 1): counter-based Gumbel noise ---------------------------------
// u in (0,1) from a 32-bit multiply-xorshift mix (MurmurHash3 finaliser family) of (seed, position,
// token id), top 23 bits centred in their cell (exact in fp32); g = -ln(-ln u) is standard Gumbel, and
// arg-max over the vocabulary of logit + g is a draw from softmax(logits).  `position` is the absolute
// position of the token being drawn, so a draw does not depend on how its position is reached.
__device__ __forceinline__ float gumbel_noise(uint32_t seed, uint32_t position, uint32_t id) {
  uint32_t x = id * 0x9E3779B1u + position * 0x85EBCA77u + seed * 0xC2B2AE3Du;
  x ^= x >> 16; x *= 0x85EBCA6Bu; x ^= x >> 13; x *= 0xC2B2AE35u; x ^= x >> 16;
  const float u = ((float)(x >> 9) + 0.5f) * (1.0f / 8388608.0f);
  return -logf(-logf(u));
}

// ---- KV cache addressing (see esp_kv in esp.h) --------------------------------------------
// Per (layer, kv head) plane of capacity*hd elements, in blocks of 32 slots stored in the order
// the matrix cores consume them (v_mfma_f32_32x32x16 A operands, 64 lanes x 8 elements each):
//   K block: [hd/16 k-steps][64 lanes][8]   lane (slot%32, half) holds features 16*step + 8*half + 0..7
//            (A operand of S^T = K Q^T: row = key, contraction over features)
//   V block: [hd/32 feature blocks][2 key-steps][64 lanes][8]   lane (feature%32, half), element j
//            holds key 16*step + 8*(j/4) + 4*half + j%4 -- the order in which the S^T accumulator
//            registers of a lane half line up as B operand of O^T = V^T P^T
// so a tile of keys is one contiguous run of bytes and every fragment is one 16-byte load per lane.
__host__ __device__ __forceinline__ size_t kv_plane(int layer, int kvh, int n_kv, int64_t cap, int hd) {
  return ((size_t)layer * n_kv + kvh) * (size_t)cap * hd;
}
__host__ __device__ __forceinline__ size_t k_off(int64_t slot, int d, int hd) {
  return (size_t)(slot >> 5) * hd * 32 + (size_t)((((d >> 4) * 64 + ((d >> 3) & 1) * 32 + (int)(slot & 31)) << 3) + (d & 7));
}
__host__ __device__ __forceinline__ size_t v_off(int64_t slot, int d, int hd) {
  const int key = (int)(slot & 31), u = key >> 4, half = (key >> 2) & 1, j = ((key >> 3) & 1) * 4 + (key & 3);
  return (size_t)(slot >> 5) * hd * 32 + (size_t)(((((d >> 5) * 2 + u) * 64 + half * 32 + (d & 31)) << 3) + j);
}

// ---- GEMM -----------------------------------------------------------------------------------
struct GemmPlan {
  int splits;        // split-K factor
  int mt;            // 32-row tiles per workgroup
  int nb;            // bf16: 1 up to 128 rows, 2 above
  int m_tiles;       // workgroup tiles along M
  int n_tiles;       // workgroup tiles along N
  int ct;            // 32-column blocks per workgroup
};
// Tiles of the bf16 kernel (esp_gemm_tile.h): row tiles and column blocks of 32 and what one costs, in ns: start and end of a round
// over the 256 CUs, a chunk of 64 of K, and how much longer a chunk takes with all CUs at it (power, L2 and HBM; with half of them,
// half of it).  Fitted to measured launches on N and K of QKV, O, gate/up and down of two model shapes, 1 to 8 splits: the first
// N_ROW_TILES, for up to 128 rows, to 1300 of 1 to 128 rows, the others to 3900 of 136 to 2112 rows.  Of the tiles and splits that were
// measured for a shape the model's choice is 0.8 % slower than the best on average, 10 % at most (17 % in one).
struct GemmTileCost { int rt, ct, start, chunk, busy; };
constexpr int N_GEMM_TILES = 23, N_ROW_TILES = 12;
constexpr GemmTileCost GEMM_TILES[N_GEMM_TILES] = {
    {1, 2, 1560, 130, 142}, {1, 4, 1770, 247, 260}, {1, 6, 2010, 381, 321}, {2, 2, 1440, 210, 88}, {2, 4, 1480, 344, 182}, {2, 6, 1640, 493, 239},
    {3, 2, 1580, 271, 68}, {3, 4, 1160, 439, 134}, {3, 6, 1560, 596, 149}, {4, 2, 1150, 326, 68}, {4, 4, 1510, 493, 158}, {4, 6, 1810, 657, 106},
    {3, 8, 3980, 582, 94}, {4, 4, 2110, 413, 124}, {4, 6, 3660, 565, 75}, {4, 8, 5010, 584, 178}, {5, 6, 4720, 589, 97}, {5, 8, 6230, 646, 218},
    {6, 6, 5400, 585, 192}, {6, 8, 6860, 710, 311}, {6, 10, 7800, 982, 206}, {8, 6, 6660, 784, 220}, {8, 8, 8130, 885, 368}};
__host__ __device__ inline int64_t tile_cost(const GemmTileCost& t, int rows, int blocks, int chunks, int splits) {
  const int64_t n = (int64_t)((rows + 32 * t.rt - 1) / (32 * t.rt)) * ((blocks + t.ct - 1) / t.ct) * splits;
  if (n == 0) return 0;
  const int64_t before = (n - 1) / 256, last = n - 256 * before, c = (chunks + splits - 1) / splits;
  return (before + 1) * t.start + c * ((before + 1) * t.chunk + t.busy * before + t.busy * last / 256);
}
GemmPlan gemm_plan(int dtype, int M, int N, int K);
// of a batch with packed rows, of whose M rows only the device knows how many are there: for two thirds of them to all
GemmPlan batch_gemm_plan(int M, int N, int K);
// split-K parts by size alone: what one round of the CUs holds of tiles of 128 columns up to 128 rows and of 160 x 256 above, each
// part with eight chunks of K or more
int round_parts(int M, int N, int K);
GemmPlan row_major_plan(int M, int N, int K);     // bf16 weights that are not packed
GemmPlan product_plan(int M, int N, int K);       // bf16, packed, for a product that is added up by a launch of its own
// is a projection's output unsplit by that (the LM head's epilogues see whole rows and are refused otherwise), and its plan
bool gemm_whole_rows(int dtype, int M, int N, int K);
GemmPlan whole_row_plan(int dtype, int M, int N, int K);
inline size_t gemm_out_elems(const GemmPlan& p, int M, int N) { return (size_t)p.splits * M * N; }
// most that a bf16 or fp32 product of up to M rows needs, a batch's among them
size_t gemm_out_elems_bound(int dtype, int M, int N, int K);
// out: fp32 [splits][M][N].  a_rows (device, may be null): physical row of A for logical row m.
// w_packed: W is in the streaming layout written by launch_pack_weight (bf16 only).
// m_live (device, may be null; bf16, packed weights and more than 128 rows only): how many of the M rows there are; row tiles
// without any are left out, rows past them are not written; the others of a row tile are computed from A's row m_live.
hipError_t launch_gemm(hipStream_t st, int dtype, const void* A, const int32_t* a_rows, const void* W,
                       float* out, int M, int N, int K, const GemmPlan& p, bool w_packed, int a_ld = 0,
                       const int32_t* m_live = nullptr);
// a_ld == 0: A is row-major [rows][K]; a_ld > 0 (bf16, unpacked weights): A is chunk-major [K/64][a_ld][64]
// fp32: act[M][ff] = silu(A Wg^T) * (A Wu^T), W = gate rows then up rows
hipError_t launch_gemm_swiglu_f32(hipStream_t st, const float* A, const float* W, float* act, int M, int ff, int K);
hipError_t launch_pack_weight(hipStream_t st, const void* src, void* dst, int N, int K);
// one-time kernel attributes of the GEMM kernels (dynamic LDS limits); call before the first launch
hipError_t gemm_prepare();
// the kernel for packed weights, a launcher per epilogue
struct TileGemm {
  const void* A; const int32_t* a_rows; const void* W; void* out;
  int M, N, K, splits, tile;               // tile: index into GEMM_TILES
  const int32_t* draw_pos; uint32_t seed; const int32_t* m_live;
  float* pairs;                            // launch_gemm_tile_both: the arg-max pairs
};
// rows of K that a 32-bit offset in bytes reaches: those of a tile have to, and all that a list (a_rows) may name
inline bool gemm_rows_fit(int64_t rows, int64_t K) { return rows * K * 2 <= (int64_t)UINT32_MAX; }
hipError_t launch_gemm_tile_out(hipStream_t st, const TileGemm& g);
hipError_t launch_gemm_tile_argmax(hipStream_t st, const TileGemm& g);
hipError_t launch_gemm_tile_swiglu(hipStream_t st, const TileGemm& g);
hipError_t launch_gemm_tile_both(hipStream_t st, const TileGemm& g);   // fp32 tile out and arg-max; tiles for up to 128 rows only
hipError_t gemm_tile_out_prepare();
hipError_t gemm_tile_argmax_prepare();
hipError_t gemm_tile_swiglu_prepare();
hipError_t gemm_tile_both_prepare();
// Tile of the gate/up projection above 128 rows, in three classes: any, by cost; one with a side of 256 (256 x 256, 192 x 256 or
// 256 x 192, by cost); and 192 x 320.  Which classes there are to choose from is said by their rounds over the 256 CUs against row
// tiles of up to 160: `rounds` in units of 10 ns, chunks x the time of one + start and epilogue (fitted to kernels before these; on its
// own it took 192 x 256 for 321 to 384 rows x 24576, where tile_cost and the clock have 192 x 192: 70 to 73 us against 65 to 66).
// For one sequence it gives way where tile_cost has another tile 6 % cheaper; up to its 1024 rows, d_ff 8192 to 18944, it is
// within 4 % otherwise.  512 x 28672 takes 95 us with 256 x 256, 576 x 24576 93 with 192 x 320, 384 x 28672 79 with 192 x 256.
// Of a batch of M block rows only the device knows how many are there: the host launches every class that a number from two
// thirds of M up asks for, the device (k_live_rows) hands the rows to the cheapest of these, and the others end at once (1.6 us).
enum GateUpTile { GU_PLAN = 0, GU_SIDE256 = 1, GU_192x320 = 2, GU_TILES = 3 };
struct GateUpRule {
  int mt = 1, chunks = 0, blocks = 0;      // row tiles of 32 where as few tiles as possible have up to five; chunks of 64 of K; column blocks of 32
  unsigned launched = 1u << GU_PLAN;       // bit t: class t is launched
  int tile[GU_TILES] = {};                 // of GEMM_TILES; up to 128 rows the first
  GemmTileCost cost[GU_TILES] = {};
  GateUpTile by_rounds(int rows) const {
    int64_t whole[GU_TILES];
    const int per[GU_TILES] = {32 * mt, 256, 192}, cols[GU_TILES] = {8, 8, 10};
    for (int t = 0; t < GU_TILES; ++t) {
      const int64_t round = t == GU_PLAN ? (int64_t)chunks * (mt >= 5 ? 90 : mt == 4 ? 80 : 74) + 650 : (int64_t)chunks * 142 + 900;
      whole[t] = ((int64_t)((rows + per[t] - 1) / per[t]) * ((blocks + cols[t] - 1) / cols[t]) + 255) / 256 * round;
    }
    const GateUpTile w = whole[GU_SIDE256] <= whole[GU_192x320] ? GU_SIDE256 : GU_192x320;
    return whole[w] * 100 < whole[GU_PLAN] * 95 ? w : GU_PLAN;
  }
  __host__ __device__ GateUpTile cheapest_launched(int rows) const {
    int best = -1;
    int64_t least = 0;
    for (int t = 0; t < GU_TILES; ++t)
      if (launched >> t & 1u) {
        const int64_t c = tile_cost(cost[t], rows, blocks, chunks, 1);
        if (best < 0 || c < least) { best = t; least = c; }
      }
    return (GateUpTile)best;
  }
};
GateUpRule gate_up_rule(int M, int ff, int K, const void* act, bool ragged);
unsigned gate_up_tiles(int M, int ff, int K, const void* act, bool ragged);   // what launch_gemm_swiglu launches
// live (device, may be null): BlockDev::n_live of a batch with packed rows
hipError_t launch_gemm_swiglu(hipStream_t st, const void* A, const void* W, void* act, int M, int ff, int K,
                              const int32_t* live = nullptr);
// the same with gate_up_rule(M, ff, K, act, live != nullptr) at hand (a layer after the other)
hipError_t launch_gate_up(hipStream_t st, const void* A, const void* W, void* act, int M, int ff, int K, const int32_t* live,
                          const GateUpRule& r);
// LM head with the arg-max taken in the GEMM epilogue (bf16, packed weights, one split)
bool gemm_argmax_supported(int dtype, int M, int N, int K, bool with_logits);
size_t gemm_argmax_scratch_floats(int M, int N);
// logits_out == NULL: arg-max of each of the M rows (out[out_index[m]]), logits never written.
// logits_out != NULL: also writes the fp32 logits [M][N]; arg-max only for the n_arg rows arg_rows[i].
hipError_t launch_gemm_argmax(hipStream_t st, const void* A, const int32_t* a_rows, const void* W, int M, int N,
                              int K, float* scratch, int32_t* out, const int32_t* out_index,
                              float* logits_out, const int32_t* arg_rows, int n_arg,
                              const int32_t* draw_pos = nullptr, uint32_t seed = 0,   // draw_pos: per GEMM row
                              const int32_t* m_live = nullptr);

// ---- elementwise / glue (esp_elementwise.hip) ----------------------------------------------
struct BlockDev {   // device-side view of esp_block + esp_kv scalars, passed by value
  int batch, rows_per_seq, k_masks, layout, anc_words;
  const int32_t *n_rows, *n_nodes, *tok, *parent, *depth, *mask_j, *attach;
  const uint64_t* anc;
  // Live rows of a ragged batch packed together (null: row m of the activations is block row m).  The kernels that use
  // them have an instantiation without (PACKED false): looking at a null pointer first cost a short launch 0.2 us.
  int32_t* packed = nullptr;
  __host__ __device__ size_t rows() const { return (size_t)batch * rows_per_seq; }
  // block row of packed row m; packed row of a block row (-1: not there); first packed row of a sequence; tree rows
  // before a sequence; [0] rows and [1] tree rows of the batch, [2 + t] rows that gate/up tile t computes (all or none)
  __host__ __device__ int32_t* live_rows() const { return packed; }
  __host__ __device__ int32_t* packed_row() const { return packed + rows(); }
  __host__ __device__ int32_t* seq_row0() const { return packed + 2 * rows(); }
  __host__ __device__ int32_t* seq_node0() const { return packed + 2 * rows() + batch; }
  __host__ __device__ int32_t* n_live() const { return packed + 2 * rows() + 2 * batch; }
  static size_t packed_ints(size_t rows, size_t batch) { return 2 * rows + 2 * batch + 2 + GU_TILES; }
};
// x, once the arguments named with it are there too: a kernel's first use of x then finds all their loads issued together.  The
// compiler loads an argument in the block that uses it, behind whatever branch comes first, and a small kernel waits for one
// line of its arguments after the other.  With this in the kernels of a layer a step of one row on 2048 keys took 3196 -> 3148
// us, of 68 rows 4084 -> 4013 (attention 11.5 -> 11.1 us a layer, each GEMM 0.1 to 0.6).  Not volatile: a statement with side
// effects would turn the uniform loads after it into vector ones.
template <typename X, typename A, typename B, typename C, typename D>
__device__ __forceinline__ X with_args(X x, A a, B b, C c, D d) {
  asm("" : "+s"(x) : "s"(a), "s"(b), "s"(c), "s"(d));
  return x;
}
template <typename X, typename A, typename B, typename C, typename D, typename E, typename F, typename G, typename H>
__device__ __forceinline__ X with_args(X x, A a, B b, C c, D d, E e, F f, G g, H h) {
  asm("" : "+s"(x) : "s"(a), "s"(b), "s"(c), "s"(d), "s"(e), "s"(f), "s"(g), "s"(h));
  return x;
}
// where row r of a sequence sits in the activations
template <bool PACKED>
__device__ __forceinline__ size_t act_row(const BlockDev& b, int seq, int r) {
  return PACKED ? (size_t)b.seq_row0()[seq] + r : (size_t)seq * b.rows_per_seq + r;
}
struct KvDev {
  void *k, *v;
  int32_t* len;
  const int32_t *base, *seq_cap;
  int64_t capacity;
  int len_bound;
};

// fills b.packed from the row counts, which only the device knows
hipError_t launch_live_rows(hipStream_t st, const BlockDev& b, const KvDev& kv, int max_nodes, const GateUpRule& gate_up);
// inputs of the projections (bf16, width a multiple of 8), of which the row behind a packed batch's live ones is zeroed
struct PackedEnd {
  bf16_t* rows[3] = {};
  int width[3] = {};
};
// gather lists for the LM head over the tree rows (max_nodes 0: not wanted): block row of node-list entry m, row of its result (-1:
// none), position of the token that follows it (len + depth + 1); row_positions (nullable): the same for every block row
struct NodeLists {
  int max_nodes = 0;
  int32_t *a_rows = nullptr, *out_rows = nullptr, *positions = nullptr, *row_positions = nullptr;
};
// h and the rotary table of every row, xn = its norm with `gain`, and the lists
hipError_t launch_embed(hipStream_t st, int dtype, const BlockDev& b, const KvDev& kv, const void* embed,
                        const void* mask_embed, float* h, int d, int vocab, float* rope_tab, int hd,
                        float theta, int32_t* status, size_t mask_seq_stride, const PackedEnd& end, const NodeLists& lists,
                        const void* gain, float eps, void* xn);
// n_live (nullable): rows there are.  packed_row (nullable): row m of xn_out comes from row packed_row[m], or is zero
hipError_t launch_residual_norm(hipStream_t st, int dtype, float* h, const float* part, int splits, int M,
                                int d, const void* gain, float eps, void* xn_out, const int32_t* n_live = nullptr,
                                const int32_t* packed_row = nullptr);
hipError_t launch_qkv_post(hipStream_t st, int dtype, const BlockDev& b, const KvDev& kv, int layer,
                           const float* part, int splits, int M, int hq, int hkv, int hd, int qk_norm,
                           const void* qg, const void* kg, float eps, const float* rope_tab, void* q_out);
// draw_pos (nullable): sample instead of arg-max -- entry m draws position draw_pos[m] with `seed`
hipError_t launch_argmax(hipStream_t st, const float* logits, size_t row_stride, const int32_t* row_map,
                         int n_rows_out, int vocab, int32_t* out, const int32_t* out_index,
                         const int32_t* draw_pos = nullptr, uint32_t seed = 0);
hipError_t launch_kv_copy(hipStream_t st, int dtype, const KvDev& kv, int layer, int n_kv, int hd,
                          int seq_base, int first_slot, int n_slots, void* k_rows, void* v_rows, int to_cache);
hipError_t launch_mask_mean(hipStream_t st, int dtype, const void* embed, const int32_t* tokens, int n, int k,
                            int d, int vocab, void* mask_embed);
hipError_t launch_mask_last_k(hipStream_t st, int dtype, const void* embed, const int32_t* tokens, int n, int k,
                              int d, int vocab, void* mask_embed);
size_t mask_gaussian_scratch_floats(int d);
hipError_t launch_mask_gaussian(hipStream_t st, int dtype, const void* embed, int vocab, int d, const float* z,
                                float shift, int k, float* scratch, size_t scratch_floats, void* mask_embed);
hipError_t launch_mask_ema(hipStream_t st, int dtype, const void* embed, const int32_t* n_emit,
                           const int32_t* emit_tok, float lambda, int k, int d, int vocab, void* mask_embed, int n_seq);

// ---- attention (esp_attn.hip) ------------------------------------------------------------------
struct AttnPlan {
  int nsplit = 1, tiles_per_split = 1;   // splits of the key range, 64-key tiles in each
  int q_tiles = 1, ct_wg = 1;            // ring kernel: workgroups per kv head and split, column tiles in each
};
AttnPlan attn_plan(int dtype, int hd, int batch, int rows_per_seq, int hq, int hkv, int len_bound);
hipError_t attn_prepare();   // one-time kernel attributes (dynamic LDS limit)
size_t attn_partial_floats(int dtype, int batch, int rows_per_seq, int hq, int hkv, int hd, const AttnPlan& p);
// what any plan for up to that many sequences and rows needs
size_t attn_partial_floats_bound(int dtype, int batch, int rows_per_seq, int hq, int hkv, int hd);
// A batch's sequences as one line of work per kv head, cut into equal shares (esp_attn.hip): how many (0: not this batch), and the
// table of the cuts, which launch_attn_cuts fills from the lengths and rows that only the device knows, for all layers at once
int attn_shares(int dtype, int hd, int batch, int rows_per_seq, int hq, int hkv, const AttnPlan& p);
size_t attn_cuts_ints(int batch);
hipError_t launch_attn_cuts(hipStream_t st, const BlockDev& b, const KvDev& kv, int hq, int hkv, const AttnPlan& p, int shares, int32_t* cuts);
// does the generic kernel merge its splits itself, groups: (row, head) pairs
bool attn_generic_merges(int hd, const AttnPlan& p, int64_t groups);
// cuts: null for a grid of equal splits.  launch_attn writes `partials`, or `out` itself where launch_attn_merge then does nothing.
hipError_t launch_attn(hipStream_t st, int dtype, const BlockDev& b, const KvDev& kv, int layer, int hq,
                       int hkv, int hd, const void* q, float* partials, const AttnPlan& p, const int32_t* cuts, void* out);
hipError_t launch_attn_merge(hipStream_t st, int dtype, const BlockDev& b, const KvDev& kv, int hq, int hkv, int hd,
                             const float* partials, const AttnPlan& p, void* out, const int32_t* cuts);

// ---- softmax + top-k (esp_topk.hip) -----------------------------------------------------------
size_t softmax_topk_scratch_floats(int rows, int vocab, int kp);
// row_map (nullable): logits row of output row r is row_map[r] (negative: 0)
hipError_t launch_softmax_topk(hipStream_t st, const float* logits, int rows, int vocab, int kp, int32_t* ids,
                               float* probs, float* scratch, const int32_t* row_map = nullptr);

// ---- tree logic (esp_tree.hip) -------------------------------------------------------------------
hipError_t tree_prepare();   // one-time kernel attributes (dynamic LDS limits)
hipError_t launch_block_from_tree(hipStream_t st, int batch, int rows_per_seq, int k, int layout, int anc_words,
                                  int32_t* n_rows, const int32_t* n_nodes, int32_t* tok, int32_t* parent,
                                  int32_t* depth, int32_t* mask_j, int32_t* attach, uint64_t* anc,
                                  int32_t* status);
hipError_t launch_verify_accept(hipStream_t st, int dtype, const BlockDev& b, const KvDev& kv,
                                const int32_t* node_argmax, int n_layers, int n_kv, int hd, int32_t* n_emit,
                                int32_t* emit_tok, int32_t* accepted_row, int32_t* star_row, int32_t* status);
hipError_t launch_mask_rows(hipStream_t st, const BlockDev& b, const int32_t* star_row, const int32_t* n_emit,
                            int32_t* a_rows, int32_t* n_lists);
hipError_t launch_build_tree(hipStream_t st, const esp_tree_params& p, int batch, const int32_t* topk_id,
                             const float* topk_p, int kp, const int32_t* n_lists, const int32_t* n_emit,
                             const int32_t* emit_tok, int rows_per_seq, int anc_words, int32_t* n_rows,
                             int32_t* n_nodes, int32_t* tok, int32_t* parent, int32_t* depth, int32_t* mask_j,
                             int32_t* attach, uint64_t* anc, int32_t* status, bool reuse);

// Events a profiling scope hands to the next bf16 GEMM launch: the launch attaches them to the kernel
// itself (hipExtLaunchKernelGGL), so they carry the kernel's own begin and end time stamps and not the
// time of two extra event commands around it.
struct LaunchEvents { hipEvent_t start = nullptr, stop = nullptr; };
extern thread_local LaunchEvents g_launch_events;

// ---- context --------------------------------------------------------------------------------------
struct esp_ctx {
  esp_model_desc m;
  const void *embed, *lm_head, *final_norm;
  std::vector<const void*> wqkv, wo, wgu, wdown, norm_attn, norm_mlp, q_norm, k_norm;
  int max_batch, max_rows;
  int64_t max_kv_len;
  hipStream_t stream;
  char* ws;
  size_t ws_bytes;
  // workspace partition
  float* h;          // [Mmax][d] fp32 residual stream
  void* xn;          // T [Mmax][d]
  void* q;           // T [Mmax][hq*hd]
  void* attn_out;    // T [Mmax][hq*hd]
  void* act;         // T [Mmax][d_ff]
  float* gemm_out;   // fp32 split-K partials of the largest layer GEMM
  float* attn_part;  // attention split partials
  // logits of all block rows left in `logits` by the last esp_tree_forward (bf16, <= 128 rows), for
  // esp_mask_topk on the same hidden states: the hidden buffer they came from and the row count
  int sample_on = 0;            // sample matching instead of greedy verification
  uint32_t sample_seed = 0;
  int32_t *idx_c, *idx_d;       // draw positions per block row / per node-list entry
  const void* lm_cache_hidden = nullptr;
  int lm_cache_rows = 0;
  // blocks that hold the rows of a fixed tree built with these parameters (esp_build_prune_tree
  // then only rewrites their tokens): identity = address of the block's token array
  bool mask_per_seq = false;    // mask vectors are [batch, k, d] (esp_set_mask_batch)
  struct StaticTreeSlot { const void* tok = nullptr; uint64_t sig = 0; };
  StaticTreeSlot static_trees[4];
  float* rope_tab;   // [Mmax][hd/2][2] cos, sin
  float* logits;     // fp32 [logits_rows][vocab]
  float* topk_scratch;
  int32_t* idx_a;    // [Mmax] gather rows
  int32_t* idx_b;    // [Mmax]
  int32_t* packed;   // packed rows of a ragged batch (BlockDev)
  int32_t* cuts;     // shares of a batch's attention
  int32_t* status;   // device status word
  size_t gemm_out_floats, attn_part_floats, logits_rows;
  // optional launch-site timing with HIP events (esp_profile_enable / esp_profile_read)
  struct ProfSpan { int site; hipEvent_t start, stop; };
  uint32_t prof_mask = 0;
  std::vector<ProfSpan> prof_open;
  std::vector<hipEvent_t> prof_pool;
  double prof_ms[ESP_SITE_COUNT] = {};
  int64_t prof_n[ESP_SITE_COUNT] = {};
};
