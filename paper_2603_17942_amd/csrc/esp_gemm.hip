// Dense projections of the decoder: out[s][M][N] (fp32 partial sums over split s) = A[M,K] * W[N,K]^T.
//
// bf16 path (the 8B-class workloads): M is the number of block rows (tens to hundreds) while W is
// hundreds of MB per layer.
//  * Weights live in HBM in a streaming layout (k_pack_weight): the 32-row x 64-k tile of a row block and
//    K-chunk is stored as [step][lane][8 values] = 4 KB contiguous in MFMA operand order, so every
//    wave-wide load covers 1 KB of consecutive addresses.  Tiles are ordered chunk-major ([chunk][row block]): at any
//    moment the waves of the whole grid, which advance through the chunks together, read one contiguous window of HBM.
//    Inside a chunk the k index is permuted identically for both operands (lane group g, step s
//    holds k = 32 g + 8 s + 0..7), which leaves the dot product unchanged.
//  * Packed weights: k_gemm_tile (esp_gemm_tile.h).  Row-major weights (esp_gemm alone): k_gemm_bf16 below.
//  * Split-K (grid z): partial sums are reduced by the consumer in split order, so a result does
//    not depend on scheduling.  The split count is a function of (N, K) up to 128 rows; above, it
//    also depends on the number of row tiles (gemm_plan), so a row's low-order bits can differ
//    between a block of 320 rows and a block of 68.
//
// fp32 path (tiny configuration, k_gemm_f32): 32 x 32 tiles on the fp32 matrix instruction, row-major weights.
#include <algorithm>
#include <type_traits>

#include "esp_gemm_common.h"

namespace {

constexpr int A_ROW_BYTES = 144;  // 128 B of bf16 + 16 B pad: conflict-free ds_read_b128 over 8 rows

// Row-major weights.  A register ring keeps D (even) chunks of weights in flight per wave; the activations of a chunk (L2
// resident, shared by the four waves through LDS) ride in a ring of the same depth and are issued together with the weights of
// the same chunk: loads retire in order, so waiting for the activations of chunk c+1 leaves the D-2 younger chunks of the
// weight stream in flight.  v_mfma_f32_32x32x16_bf16; LDS fragment reads are double-buffered one MFMA step ahead.
template <int MT, int NB, int D>
__device__ __forceinline__ void gemm_bf16_body(unsigned char* lds, const bf16_t* __restrict__ A,
                                               const int32_t* __restrict__ a_rows, const bf16_t* __restrict__ W,
                                               float* __restrict__ out, int M, int N, int K, int splits,
                                               int m_tiles, int n_tiles, int a_ld) {
  // XCD-aware logical id: consecutive hardware ids go to different XCDs, so give each XCD a
  // contiguous range of tiles (tiles sharing weight rows then share an L2).
  const int total = m_tiles * n_tiles * splits;
  const int per_xcd = (total + 7) >> 3;
  const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (logical >= total) return;
  const int mi = logical % m_tiles;
  const int ni = (logical / m_tiles) % n_tiles;
  const int z = logical / (m_tiles * n_tiles);

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int lr = lane & 31, lg = lane >> 5;
  const int m0 = mi * (MT * 32);                 // first row of the workgroup tile
  const int n0 = ni * (128 * NB) + wave * (32 * NB);

  const int chunks = K / KC;
  const int cps = (chunks + splits - 1) / splits;
  const int c_begin = z * cps;
  const int c_end = min(chunks, c_begin + cps);

  f32x16_t acc[MT][NB];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // weight pointers (clamped: out-of-range column blocks are computed but never stored)
  const u32x4_t* wp[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) wp[nb] = reinterpret_cast<const u32x4_t*>(W + (size_t)min(n0 + nb * 32 + lr, N - 1) * K + 32 * lg);
  constexpr size_t W_CHUNK = KC * 2 / 16;               // u32x4_t between chunks of a lane's stream

  // activation staging: thread handles MT pieces of 16 B; piece p -> row p/8, 16-byte column p%8
  const bf16_t* ap[MT];
  int a_lds[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    int p = tid + 256 * i;
    int r = p >> 3, c16 = p & 7;
    int m = min(m0 + r, M - 1);
    if (a_rows) m = max(a_rows[m], 0);
    ap[i] = A + (a_ld > 0 ? (size_t)m * KC : (size_t)m * K) + c16 * 8;
    a_lds[i] = r * A_ROW_BYTES + c16 * 16;
  }
  // activations: row-major [M][K] (a_ld == 0), or chunk-major [K/64][a_ld][64] where the rows of
  // one 64-wide k chunk are contiguous (row-major puts them 2K bytes apart, which lands every row
  // of a chunk on the same L2 channel when all workgroups walk the chunks in step)
  const size_t a_cs = a_ld > 0 ? (size_t)a_ld * KC : (size_t)KC;
  constexpr int A_BUF = MT * 32 * A_ROW_BYTES;

  u32x4_t wreg[D][NB][4];
  u32x4_t areg[D][MT];

  // Every group of D chunks but the last refills the ring with the same loads (chunk indices past the
  // split are clamped to its last chunk, an L2 hit, and their activations are zeroed so they add
  // nothing): with a fixed number of loads in flight the compiler can wait for exactly the chunk it
  // needs.  The last group is code of its own that loads nothing: its refills would be D chunks of
  // repeated reads a workgroup (the O projection has 8 of its own), waited for by nobody but queued
  // before the next kernel's.  With and without them, both in one run: step of one row 3562 -> 3535 us (runs of one side
  // differ by 1.8 %), 30 rows 3782 -> 3716, 68 rows 4709 -> 4658, 101 rows of the Qwen3 shape 5978 -> 5904.  (Deeper
  // rings, 8 chunks at <= 64 rows and 6 above, were slower by 2 to 5 %.)
  const int c_last = max(c_end - 1, c_begin);
  const u32x4_t zero4 = {0u, 0u, 0u, 0u};
  // prologue: chunks c_begin .. c_begin+D-1
#pragma unroll
  for (int u = 0; u < D; ++u) {
    const int c = c_begin + u;
    const int cc = min(c, c_last);
#pragma unroll
    for (int i = 0; i < MT; ++i) areg[u][i] = *reinterpret_cast<const u32x4_t*>(ap[i] + (size_t)cc * a_cs);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int s = 0; s < 4; ++s) wreg[u][nb][s] = wp[nb][(size_t)cc * W_CHUNK + s];
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
    *reinterpret_cast<u32x4_t*>(lds + a_lds[i]) = c_begin < c_end ? areg[0][i] : zero4;
  __syncthreads();

  const int n_iter = (c_end - c_begin + D - 1) / D;   // groups of D chunks, the last one zero-padded
  auto group = [&](int it, auto refill) {
    constexpr bool REFILL = decltype(refill)::value;
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int c = c_begin + it * D + u;
      const int buf = u & 1;                            // D is even
      const unsigned char* abase = lds + buf * A_BUF + lr * A_ROW_BYTES + 64 * lg;
      // Fragment reads run one MFMA step ahead and are pinned between the MFMA groups (scheduling
      // barriers), so each read has MT*NB MFMAs of cover before its first use.
      bf16x8_t af[2][MT];
#pragma unroll
      for (int i = 0; i < MT; ++i) af[0][i] = *reinterpret_cast<const bf16x8_t*>(abase + i * 32 * A_ROW_BYTES);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          if (s < 3)
            af[(s + 1) & 1][i] = *reinterpret_cast<const bf16x8_t*>(abase + i * 32 * A_ROW_BYTES + 16 * (s + 1));
          if constexpr (REFILL) {
            // refill of ring slot u with chunk c+D, one load per MFMA group (a burst after the
            // MFMAs would hold the wave at the memory pipeline's address queue while the matrix
            // cores idle): the activation registers are free (stored to LDS a chunk ago), the
            // weight registers of step s-1 were consumed by the previous step
            const int cc = min(c + D, c_last);
            if (s == 0) areg[u][i] = *reinterpret_cast<const u32x4_t*>(ap[i] + (size_t)cc * a_cs);
            else if (i < NB) wreg[u][i][s - 1] = wp[i][(size_t)cc * W_CHUNK + s - 1];
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            bf16x8_t bfr = __builtin_bit_cast(bf16x8_t, wreg[u][nb][s]);
            acc[i][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[s & 1][i], bfr, acc[i][nb], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (!REFILL && u == D - 1) return;                // nothing follows
      // activations of chunk c+1 (ring slot u+1) -> the other LDS buffer
#pragma unroll
      for (int i = 0; i < MT; ++i)
        *reinterpret_cast<u32x4_t*>(lds + (buf ^ 1) * A_BUF + a_lds[i]) =
            c + 1 < c_end ? areg[(u + 1) % D][i] : zero4;   // zeroed at use, not at load
      // the last step's weight registers of ring slot u
      if constexpr (REFILL) {
        const int cc = min(c + D, c_last);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) wreg[u][nb][3] = wp[nb][(size_t)cc * W_CHUNK + 3];
      }
      __syncthreads();
    }
  };
  for (int it = 0; it + 1 < n_iter; ++it) group(it, std::true_type{});
  if (n_iter > 0) group(n_iter - 1, std::false_type{});
  __syncthreads();                                      // the epilogues reuse the LDS

  // epilogue: lane holds column n, rows 8*(v/4) + 4*lg + v%4 of each 32x32 tile
  float* o = out + (size_t)z * M * N;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int n = n0 + nb * 32 + lr;
    if (n0 + nb * 32 < N) {
#pragma unroll
      for (int i = 0; i < MT; ++i) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          int m = m0 + i * 32 + 8 * (v >> 2) + 4 * lg + (v & 3);
          if (m < M) o[(size_t)m * N + n] = acc[i][nb][v];
        }
      }
    }
  }
}

// Two entry points over the same body.  The small-tile one leaves occupancy to the compiler.  The large-tile one tells it that
// one wave per SIMD is all it will ever get, so registers go to prefetching.
template <int MT, int NB>
__global__ __launch_bounds__(256) void k_gemm_bf16(const bf16_t* __restrict__ A, const int32_t* __restrict__ a_rows,
                                                   const bf16_t* __restrict__ W, float* __restrict__ out, int M,
                                                   int N, int K, int splits, int m_tiles, int n_tiles, int a_ld) {
  extern __shared__ __align__(16) unsigned char lds[];   // 2 buffers of MT*32 rows * A_ROW_BYTES
  gemm_bf16_body<MT, NB, 4>(lds, A, a_rows, W, out, M, N, K, splits, m_tiles, n_tiles, a_ld);
}

template <int MT, int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_gemm_bf16_big(
    const bf16_t* __restrict__ A, const int32_t* __restrict__ a_rows, const bf16_t* __restrict__ W,
    float* __restrict__ out, int M, int N, int K, int splits, int m_tiles, int n_tiles, int a_ld) {
  extern __shared__ __align__(16) unsigned char lds[];
  gemm_bf16_body<MT, NB, 2>(lds, A, a_rows, W, out, M, N, K, splits, m_tiles, n_tiles, a_ld);
}

// ---- fp32: one 32 x 32 tile per workgroup, its eight waves split K (v_mfma_f32_32x32x2_f32) --------
// The fp32 models are small (256 x 256 to 4096 x 256 weights): latency is the bound, so a tile is as
// small as a matrix instruction, every wave has an eighth of K to itself and issues its loads up front
// (F32_U chunks of 8 k in flight, no barrier in the loop), and the eight partial tiles meet once in LDS,
// added in wave order.  Within a chunk the k index is permuted alike for both operands (lane half g
// holds k = 8 c + 4 g + 0..3), so a lane's operands of four matrix instructions are one 16-byte load.
// K not a multiple of 4, or rows that are not 16-byte aligned (VEC false): the same with scalar loads.
// MI355X, a step of the 2-layer d = 256 model at 60 rows (nine of these launches): 678 -> 176 us against a
// 64 x 64 tile walked in 16-deep steps through LDS, each step exposing a memory latency (39 to 123 us
// a launch).
constexpr int F32_WAVES = 8, F32_U = 4;

template <bool VEC>
__device__ __forceinline__ f32x4_t f32_piece(const float* __restrict__ row, int k, int K) {
  f32x4_t v = {0.f, 0.f, 0.f, 0.f};
  if (VEC) {
    if (k < K) v = *reinterpret_cast<const f32x4_t*>(row + k);   // K % 4 == 0: all or nothing
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k + e < K) v[e] = row[k + e];
  }
  return v;
}

// SWIGLU: the 32 weight rows of a tile are 16 gate features and the 16 up features of the same number (N rows behind), and
// silu(gate) * up goes out, [M][N]: a launch less and twice the workgroups of a tile of each, bit for bit what the product and a
// kernel for the activation after it gave.  60 x (2 x 688) x 256: 6.0 + 2.8 -> 6.2 us; 8.9 with a gate tile and an up tile in a
// workgroup, of eight waves or of sixteen.
template <bool VEC, bool SWIGLU>
__global__ __launch_bounds__(64 * F32_WAVES) void k_gemm_f32(const float* __restrict__ A, const int32_t* __restrict__ a_rows,
                                                             const float* __restrict__ W, float* __restrict__ out, int M,
                                                             int N, int K) {
  __shared__ float part[F32_WAVES][16][64];
  constexpr int COLS = SWIGLU ? 16 : 32;
  const int m0 = blockIdx.y * 32, n0 = blockIdx.x * COLS;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lr = lane & 31, lg = lane >> 5;
  int m = min(m0 + lr, M - 1);                      // clamped rows and columns are computed, never stored
  if (a_rows) m = max(a_rows[m], 0);
  const float* ar = A + (size_t)m * K;
  const float* wr = W + (size_t)(min(n0 + lr % COLS, N - 1) + lr / COLS * N) * K;
  const int chunks = (K + 7) >> 3;
  const int mine = (chunks - wave + F32_WAVES - 1) / F32_WAVES;   // chunks wave, wave + 8, ...
  f32x16_t acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  f32x4_t a[2][F32_U], w[2][F32_U];
  auto load = [&](int buf, int i0) {
#pragma unroll
    for (int u = 0; u < F32_U; ++u) {
      const int k = (i0 + u < mine ? (wave + F32_WAVES * (i0 + u)) * 8 : K) + 4 * lg;   // past the share: zeros
      a[buf][u] = f32_piece<VEC>(ar, k, K);
      w[buf][u] = f32_piece<VEC>(wr, k, K);
    }
  };
  load(0, 0);
  for (int i0 = 0; i0 < mine; i0 += 2 * F32_U) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      load(b ^ 1, i0 + (b + 1) * F32_U);
#pragma unroll
      for (int u = 0; u < F32_U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[b][u][e], w[b][u][e], acc, 0, 0, 0);
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) part[wave][v][lane] = acc[v];
  __syncthreads();
  for (int e = tid; e < 32 * COLS; e += 64 * F32_WAVES) {
    const int v = e / (2 * COLS), c = e % COLS, h = e / COLS % 2, l = 32 * h + c;
    float sum = part[0][v][l];
#pragma unroll
    for (int q = 1; q < F32_WAVES; ++q) sum += part[q][v][l];
    if (SWIGLU) {
      float up = part[0][v][l + COLS];
#pragma unroll
      for (int q = 1; q < F32_WAVES; ++q) up += part[q][v][l + COLS];
      sum = sum / (1.0f + expf(-sum)) * up;
    }
    const int mo = m0 + 8 * (v >> 2) + 4 * h + (v & 3), no = n0 + c;
    if (mo < M && no < N) out[(size_t)mo * N + no] = sum;
  }
}

// row-major [N][K] -> tiles of 32 rows x 64 k stored as [chunk][row block][step][lane][8]
__global__ void k_pack_weight(const bf16_t* __restrict__ src, bf16_t* __restrict__ dst, int N, int K) {
  const size_t piece = (size_t)blockIdx.x * blockDim.x + threadIdx.x;   // one 16-byte piece
  const size_t total = (size_t)N * K / 8;
  if (piece >= total) return;
  const int chunks = K / KC;
  const int lane = piece & 63, s = (piece >> 6) & 3;
  const size_t tile = piece >> 8;
  const int nblk = N >> 5;
  const int blk = (int)(tile % nblk);
  const int c = (int)(tile / nblk);
  const int n = blk * 32 + (lane & 31);
  const int k = c * KC + 32 * (lane >> 5) + 8 * s;
  reinterpret_cast<uint4*>(dst)[piece] = *reinterpret_cast<const uint4*>(src + (size_t)n * K + k);
}

template <int MT, int NB>
hipError_t launch_bf16(hipStream_t st, const void* A, const int32_t* a_rows, const void* W, float* out, int M, int N, int K, int splits,
                       int a_ld) {
  const int m_tiles = (M + 32 * MT - 1) / (32 * MT), n_tiles = (N + 128 * NB - 1) / (128 * NB);
  const auto kern = MT * NB >= 8 ? k_gemm_bf16_big<MT, NB> : k_gemm_bf16<MT, NB>;
  launch_kernel(kern, dim3((m_tiles * n_tiles * splits + 7) / 8 * 8), dim3(256), 2 * (size_t)MT * 32 * A_ROW_BYTES, st, (const bf16_t*)A,
                a_rows, (const bf16_t*)W, out, M, N, K, splits, m_tiles, n_tiles, a_ld);
  return hipGetLastError();
}

// row tiles of 32 where as few tiles as possible have up to five
int even_row_tiles(int M) {
  const int t = (M + 31) / 32, n = (t + 4) / 5;
  return (t + n - 1) / n;
}

// of GEMM_TILES: the tile of a plan
int tile_index(const GemmPlan& p) {
  for (int t = p.nb == 1 ? 0 : N_ROW_TILES; t < N_GEMM_TILES; ++t)
    if (GEMM_TILES[t].rt == p.mt && GEMM_TILES[t].ct == p.ct) return t;
  return -1;
}

// Tile and split-K parts of a launch of more than 128 rows: the cheapest by GEMM_TILES, plus what the partials cost on their way
// out and in (1 us for 4 MB).  There are `fewest` parts at least (gemm_plan); more of them fit one round of the CUs and have eight
// chunks of K or more.  Of a batch, over numbers of rows from two thirds of M up.
GemmPlan tile_plan(int M, int N, int K, int fewest, int most, bool batch) {
  const int rows = (M + 31) / 32 * 32, blocks = (N + 31) / 32, chunks = std::max(K / KC, 1), at[3] = {rows, rows * 5 / 6, rows * 2 / 3};
  const int max_s = std::max(fewest, std::min(most, chunks / 8));
  GemmPlan best{};
  int64_t least = -1;
  for (int t = N_ROW_TILES; t < N_GEMM_TILES; ++t) {
    const GemmTileCost& c = GEMM_TILES[t];
    const int m_tiles = (M + 32 * c.rt - 1) / (32 * c.rt), n_tiles = (blocks + c.ct - 1) / c.ct;
    for (int s = fewest; s <= max_s; ++s) {
      if (s > fewest && (int64_t)m_tiles * n_tiles * s > 256) break;
      const int cps = (chunks + s - 1) / s;
      if (s > fewest && (chunks + cps - 1) / cps != s) continue;   // the same parts as with fewer
      int64_t cost = 0;
      for (int i = 0; i < (batch ? 3 : 1); ++i) cost += tile_cost(c, at[i], blocks, chunks, s) + (int64_t)s * at[i] * N / 1000;
      if (least < 0 || cost < least) {
        least = cost;
        best.splits = s; best.mt = c.rt; best.nb = 2; best.m_tiles = m_tiles; best.n_tiles = n_tiles; best.ct = c.ct;
      }
    }
  }
  return best;
}

// Up to 128 rows: one row tile.  The parts are a function of (N, K), those of 128 rows: a row's sums then do not depend on how
// many rows there are beside it.  There are `fewest` at least (gemm_plan; 5, 8 and 8 for QKV, O and down of the 8B shapes), and a part
// beyond that costs its consumer 0.6 us beside its bytes.  The columns are what is cheapest for the parts.  fewest_ct: 4 where pairs
// for every 128 columns have been reserved.
GemmPlan row_plan(int M, int N, int K, int fewest, int most, int fewest_ct) {
  const int blocks = (N + 31) / 32, chunks = std::max(K / KC, 1), rt = (M + 31) / 32;
  const int max_s = std::max(fewest, std::min(most, chunks / 8));
  GemmPlan best{};
  for (int pass = 0; pass < 2; ++pass) {                 // the parts with four row tiles, then the columns with rt
    const int pass_rt = pass ? rt : 4, s0 = pass ? best.splits : fewest, s1 = pass ? best.splits : max_s;
    int64_t least = -1;
    for (int t = 0; t < N_ROW_TILES; ++t) {
      const GemmTileCost& c = GEMM_TILES[t];
      if (c.rt != pass_rt || c.ct < fewest_ct) continue;
      const int n_tiles = (blocks + c.ct - 1) / c.ct;
      for (int s = s0; s <= s1; ++s) {
        if (s > s0 && n_tiles * s > 256) break;
        const int cps = (chunks + s - 1) / s;
        if (s > s0 && (chunks + cps - 1) / cps != s) continue;
        const int64_t cost = tile_cost(c, 32 * pass_rt, blocks, chunks, s) + (int64_t)s * (32 * pass_rt * N / 1000 + 600);
        if (least < 0 || cost < least) {
          least = cost;
          best.splits = s; best.mt = rt; best.nb = 1; best.m_tiles = 1; best.n_tiles = n_tiles; best.ct = c.ct;
        }
      }
    }
  }
  return best;
}

}  // namespace

thread_local LaunchEvents g_launch_events;

hipError_t gemm_prepare() {
  hipError_t e = gemm_tile_out_prepare();
  if (e == hipSuccess) e = gemm_tile_argmax_prepare();
  if (e == hipSuccess) e = gemm_tile_swiglu_prepare();
  if (e == hipSuccess) e = gemm_tile_both_prepare();
  return e;
}

// No fewer parts than round_parts: a part is one running fp32 sum, whose error grows with the root of its terms.  Chosen by time
// alone (2, 4 and 4 parts for QKV, O and down up to 128 rows, 4 and 5 for QKV and O at 320) the products' error against 64 bits was up to
// 1.62 times as large (QKV up to 128 rows 2.72e-7, now 1.68e-7).  The time of a step that way and this way: one row 3139 and 3178 us,
// 68 rows 3973 and 4063, 101 rows of the Qwen3 shape 5149 and 5335, 320 rows 6845 and 7068, 576 rows of the Qwen3 shape 10828 and 10723.
GemmPlan gemm_plan(int dtype, int M, int N, int K) {
  GemmPlan p;
  if (dtype == ESP_F32) {
    p.splits = 1; p.mt = 1; p.nb = 1; p.m_tiles = (M + 31) / 32; p.n_tiles = (N + 31) / 32; p.ct = 1;
    return p;
  }
  return M > 128 ? tile_plan(M, N, K, round_parts(M, N, K), 8, false) : row_plan(M, N, K, round_parts(M, N, K), 8, 2);
}

GemmPlan batch_gemm_plan(int M, int N, int K) { return tile_plan(M, N, K, round_parts(M, N, K), 8, true); }

int round_parts(int M, int N, int K) {
  const int m_tiles = M <= 128 ? 1 : ((M + 31) / 32 + 4) / 5, n_tiles = M <= 128 ? (N + 127) / 128 : (N + 255) / 256;
  return std::max(1, std::min(std::min(256 / (m_tiles * n_tiles), K / (KC * 8)), 8));
}
// Row-major weights: tiles of their own kernel, 128 columns up to 128 rows and 256 above.  With the parts of the packed weights' kernel,
// whose tiles are narrower, up to half of the CUs had none: 68 x 6144 x 4096 23.1 against 34.3 us, 128 x 4096 x 14336 42.0 against
// 65.8, 512 x 4096 x 4096 42.4 against 62.4.
GemmPlan row_major_plan(int M, int N, int K) {
  GemmPlan p;
  p.splits = round_parts(M, N, K);
  p.nb = M > 128 ? 2 : 1;
  p.mt = M > 128 ? even_row_tiles(M) : (M + 31) / 32;
  p.ct = 4 * p.nb;
  p.m_tiles = (M + 32 * p.mt - 1) / (32 * p.mt); p.n_tiles = (N + 32 * p.ct - 1) / (32 * p.ct);
  return p;
}
bool gemm_whole_rows(int dtype, int M, int N, int K) { return dtype == ESP_F32 || round_parts(M, N, K) == 1; }

GemmPlan whole_row_plan(int dtype, int M, int N, int K) {
  if (dtype == ESP_BF16) return M > 128 ? tile_plan(M, N, K, 1, 1, false) : row_plan(M, N, K, 1, 1, 4);
  return gemm_plan(dtype, M, N, K);
}

// Of a product on its own, whose parts nobody adds up but a launch more: not split where a round of the CUs had no room for it; above
// 128 rows unless that saves the launch (5 us) and its traffic (4 TB/s) too.  Whole and in two parts with their sum: 101 x 24576 x
// 4096 42 and 47.5 us, 128 x 18944 x 2048 24.8 and 31, 180 x 28672 x 4096 59 and 72, 1344 x 4096 x 4096 50 and 56.5.
GemmPlan product_plan(int M, int N, int K) {
  const GemmPlan p = gemm_plan(ESP_BF16, M, N, K);
  if (p.splits == 1 || !gemm_whole_rows(ESP_BF16, M, N, K)) return p;
  if (M <= 128) return row_plan(M, N, K, 1, 1, 2);
  const GemmPlan whole = whole_row_plan(ESP_BF16, M, N, K);
  const int blocks = (N + 31) / 32, chunks = std::max(K / KC, 1);
  const int64_t add = 5000 + (int64_t)(p.splits + 1) * M * N / 1000;
  return tile_cost(GEMM_TILES[tile_index(whole)], M, blocks, chunks, 1) <= tile_cost(GEMM_TILES[tile_index(p)], M, blocks, chunks, p.splits) + add ? whole : p;
}

size_t gemm_out_elems_bound(int dtype, int M, int N, int K) {
  size_t most = gemm_out_elems(gemm_plan(dtype, M, N, K), M, N);
  if (dtype != ESP_BF16) return most;
  for (int m = 32; m < M + 32; m += 32) {                // plans are the same for the rows of a tile of 32
    const int rows = std::min(m, M);
    most = std::max(most, gemm_out_elems(gemm_plan(dtype, rows, N, K), rows, N));
    if (rows > 128) most = std::max(most, gemm_out_elems(batch_gemm_plan(rows, N, K), rows, N));
  }
  return most;
}

namespace {

// arg-max over the per-tile partials written by the AMAX epilogue: one workgroup per row
__global__ __launch_bounds__(256) void k_argmax_tiles(const float* __restrict__ part, int n_tiles, int M,
                                                      const int32_t* __restrict__ row_map, int32_t* __restrict__ out,
                                                      const int32_t* __restrict__ out_index) {
  __shared__ float sv[4];
  __shared__ int si[4];
  const int dst = out_index ? out_index[blockIdx.x] : (int)blockIdx.x;
  if (dst < 0) return;
  const int m = row_map ? max(row_map[blockIdx.x], 0) : (int)blockIdx.x;   // row of the pair table
  float best = -INFINITY;
  int bi = 0x7fffffff;
  for (int t = threadIdx.x; t < n_tiles; t += 256) {
    float v = part[((size_t)t * M + m) * 2];
    int i = __float_as_int(part[((size_t)t * M + m) * 2 + 1]);
    if (v > best || (v == best && i < bi)) { best = v; bi = i; }
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

}  // namespace

// LM head with the arg-max taken in the GEMM epilogue (bf16, packed weights): scratch holds
// n_tiles * M (value, column) pairs; out[out_index[m]] = arg-max of row m.  Up to 128 rows the
// logits of all rows can be written as well (logits_out); above, the large-tile kernel takes the
// arg-max only and the [rows, vocab] logits are never written.
bool gemm_argmax_supported(int dtype, int M, int N, int K, bool with_logits) {
  return dtype == ESP_BF16 && gemm_whole_rows(dtype, M, N, K) && (M <= 128 || !with_logits);
}
size_t gemm_argmax_scratch_floats(int M, int N) { return (size_t)((N + 127) / 128) * M * 2; }

hipError_t launch_gemm_argmax(hipStream_t st, const void* A, const int32_t* a_rows, const void* W, int M, int N,
                              int K, float* scratch, int32_t* out, const int32_t* out_index,
                              float* logits_out, const int32_t* arg_rows, int n_arg, const int32_t* draw_pos,
                              uint32_t seed, const int32_t* m_live) {
  const GemmPlan p = whole_row_plan(ESP_BF16, M, N, K);
  // without logits_out: pairs only (the logits are never written); with it: the fp32 logits of all M
  // rows as well
  if (logits_out && p.nb != 1) return hipErrorInvalidValue;
  const TileGemm g{A, a_rows, W, logits_out, M, N, K, 1, tile_index(p), draw_pos, seed, m_live, scratch};
  const hipError_t e = logits_out ? launch_gemm_tile_both(st, g) : launch_gemm_tile_argmax(st, g);
  if (e != hipSuccess) return e;
  // out[out_index[i]] = arg-max of row arg_rows[i] (or of row i), i < n_arg
  hipLaunchKernelGGL(k_argmax_tiles, dim3(n_arg), dim3(256), 0, st, scratch, p.n_tiles, M, arg_rows, out, out_index);
  return hipGetLastError();
}

GateUpRule gate_up_rule(int M, int ff, int K, const void* act, bool ragged) {
  GateUpRule r;
  r.mt = even_row_tiles(M); r.chunks = K / KC; r.blocks = (2 * ff) >> 5;
  if (M <= 128) {
    r.tile[GU_PLAN] = tile_index(row_plan(M, 2 * ff, K, 1, 1, 2));
    return r;
  }
  if ((uintptr_t)act % 16 == 0 && ff % 8 == 0) {         // (the wide classes' results are stored 16 bytes at a time)
    r.launched = 1u << r.by_rounds(M);
    if (ragged)                                          // (every tile ends at a multiple of 32 rows)
      for (int rows = (2 * M / 3) & ~31; rows < M; rows += 32) r.launched |= 1u << r.by_rounds(std::max(rows, 1));
  }
  // tiles of the classes: any; a side of 256; 192 x 320
  static_assert(GEMM_TILES[19].ct == 8 && GEMM_TILES[21].rt == 8 && GEMM_TILES[22].rt == 8 && GEMM_TILES[20].ct == 10, "");
  const unsigned of[GU_TILES] = {(1u << N_GEMM_TILES) - (1u << N_ROW_TILES), 1u << 19 | 1u << 21 | 1u << 22, 1u << 20};
  // for M rows, or of a batch for any number from 0.6 M up, each of which takes the cheapest of the tiles launched; all M rows
  // may take 3 % longer than with the best for them
  constexpr int MOST = 5;
  const int n = ragged ? MOST : 1;
  int64_t cost[N_GEMM_TILES][MOST];
  for (int t = 0; t < N_GEMM_TILES; ++t)
    for (int i = 0; i < n; ++i) cost[t][i] = tile_cost(GEMM_TILES[t], std::max(M * (10 - i) / 10, 1), r.blocks, r.chunks, 1);
  int64_t least = -1, best_full = -1;
  for (int c = 0; c < GU_TILES; ++c)
    for (int t = 0; t < N_GEMM_TILES; ++t)
      if ((r.launched >> c & 1u) && (of[c] >> t & 1u) && (best_full < 0 || cost[t][0] < best_full)) best_full = cost[t][0];
  if (!ragged) {
    int64_t best = cost[N_ROW_TILES][0];
    for (int t = N_ROW_TILES; t < N_GEMM_TILES; ++t) best = std::min(best, cost[t][0]);
    if (best_full * 100 > best * 106) { r.launched = 1u << GU_PLAN; best_full = best; }
  }
  int pick[GU_TILES];
  auto choose = [&](auto&& self, int c) -> void {
    if (c < GU_TILES) {
      for (int t = 0; t < N_GEMM_TILES; ++t)
        if (r.launched >> c & 1u ? of[c] >> t & 1u : t == 20) {       // (a class that is not launched: whichever)
          pick[c] = t;
          self(self, c + 1);
        }
      return;
    }
    int64_t sum = 0;
    for (int i = 0; i < n; ++i) {
      int64_t lowest = -1;
      for (int k = 0; k < GU_TILES; ++k)
        if (r.launched >> k & 1u)
          if (lowest < 0 || cost[pick[k]][i] < lowest) lowest = cost[pick[k]][i];
      if (i == 0 && lowest * 100 > best_full * 103) return;
      sum += lowest;
    }
    if (least < 0 || sum < least) {
      least = sum;
      for (int k = 0; k < GU_TILES; ++k) { r.tile[k] = pick[k]; r.cost[k] = GEMM_TILES[pick[k]]; }
    }
  };
  choose(choose, 0);
  return r;
}
unsigned gate_up_tiles(int M, int ff, int K, const void* act, bool ragged) { return gate_up_rule(M, ff, K, act, ragged).launched; }

// Fused gate/up projection + SwiGLU (bf16, packed weights whose rows alternate in blocks of 32
// between gate and up): act[M][ff] = silu(A Wg^T) * (A Wu^T), one pass over K per workgroup.
hipError_t launch_gemm_swiglu(hipStream_t st, const void* A, const void* W, void* act, int M, int ff, int K, const int32_t* live) {
  return launch_gate_up(st, A, W, act, M, ff, K, live, gate_up_rule(M, ff, K, act, live != nullptr));
}
hipError_t launch_gate_up(hipStream_t st, const void* A, const void* W, void* act, int M, int ff, int K, const int32_t* live,
                          const GateUpRule& r) {
  if (M <= 0) return hipSuccess;
  const unsigned tiles = r.launched;
  TileGemm g{A, nullptr, W, act, M, 2 * ff, K, 1, 0, nullptr, 0u, live, nullptr};
  if ((tiles & (tiles - 1)) == 0) {
    g.tile = r.tile[__builtin_ctz(tiles)];
    return launch_gemm_tile_swiglu(st, g);
  }
  const LaunchEvents span = g_launch_events;             // a profiling span covers all of them
  for (int t = 0; t < GU_TILES; ++t) {
    if (!((tiles >> t) & 1u)) continue;
    g_launch_events = LaunchEvents{(tiles & ((1u << t) - 1)) == 0 ? span.start : nullptr, (tiles >> (t + 1)) == 0 ? span.stop : nullptr};
    g.tile = r.tile[t];
    g.m_live = live + 2 + t;
    const hipError_t e = launch_gemm_tile_swiglu(st, g);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_gemm_swiglu_f32(hipStream_t st, const float* A, const float* W, float* act, int M, int ff, int K) {
  const bool vec = K % 4 == 0 && (((uintptr_t)A | (uintptr_t)W) & 15) == 0;
  hipLaunchKernelGGL((vec ? k_gemm_f32<true, true> : k_gemm_f32<false, true>), dim3((ff + 15) / 16, (M + 31) / 32), dim3(64 * F32_WAVES), 0, st,
                     A, (const int32_t*)nullptr, W, act, M, ff, K);
  return hipGetLastError();
}

hipError_t launch_pack_weight(hipStream_t st, const void* src, void* dst, int N, int K) {
  size_t pieces = (size_t)N * K / 8;
  hipLaunchKernelGGL(k_pack_weight, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, st, (const bf16_t*)src,
                     (bf16_t*)dst, N, K);
  return hipGetLastError();
}

hipError_t launch_gemm(hipStream_t st, int dtype, const void* A, const int32_t* a_rows, const void* W,
                       float* out, int M, int N, int K, const GemmPlan& p, bool w_packed, int a_ld, const int32_t* m_live) {
  if (M <= 0) return hipSuccess;
  if (dtype == ESP_F32) {
    const bool vec = K % 4 == 0 && (((uintptr_t)A | (uintptr_t)W) & 15) == 0;
    hipLaunchKernelGGL((vec ? k_gemm_f32<true, false> : k_gemm_f32<false, false>), dim3(p.n_tiles, p.m_tiles), dim3(64 * F32_WAVES), 0, st,
                       (const float*)A, a_rows, (const float*)W, out, M, N, K);
    return hipGetLastError();
  }
  if (w_packed) {
    if (a_ld) return hipErrorInvalidValue;
    return launch_gemm_tile_out(st, {A, a_rows, W, out, M, N, K, p.splits, tile_index(p), nullptr, 0u, m_live, nullptr});
  }
  if (p.nb == 1) switch (p.mt) {
    case 1: return launch_bf16<1, 1>(st, A, a_rows, W, out, M, N, K, p.splits, a_ld);
    case 2: return launch_bf16<2, 1>(st, A, a_rows, W, out, M, N, K, p.splits, a_ld);
    case 3: return launch_bf16<3, 1>(st, A, a_rows, W, out, M, N, K, p.splits, a_ld);
    case 4: return launch_bf16<4, 1>(st, A, a_rows, W, out, M, N, K, p.splits, a_ld);
  }
  if (p.nb == 2) switch (p.mt) {
    case 3: return launch_bf16<3, 2>(st, A, a_rows, W, out, M, N, K, p.splits, a_ld);
    case 4: return launch_bf16<4, 2>(st, A, a_rows, W, out, M, N, K, p.splits, a_ld);
    case 5: return launch_bf16<5, 2>(st, A, a_rows, W, out, M, N, K, p.splits, a_ld);
  }
  return hipErrorInvalidValue;
}
