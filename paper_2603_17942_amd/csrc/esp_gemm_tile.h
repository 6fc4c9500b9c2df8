// GEMM of the bf16 models on packed weights: out[s][M][N] = A[M,K] * W[N,K]^T, with four epilogues.
//
// Above 128 rows what bounds it is the chip's power: with the matrix cores busy the clock falls to 1.6 to 1.9 of 2.4 GHz, so the
// kernel that spends the least energy per flop is the fastest.  Sustained on all CUs with operands from LDS, random data: 1.69 PFLOP/s with
// v_mfma_f32_32x32x16_bf16 (1.79 without the LDS reads), 1.88 (2.07) with v_mfma_f32_16x16x32_bf16, which reads and writes an
// accumulator half as often.  Hence 16x16x32; four waves in 2 x 2, one per SIMD with all 512 registers, which read fewer
// fragment bytes per flop than four side by side; both operands global -> LDS without a register hop; consecutive MFMAs that
// share an operand.  Accumulators in the 256 AGPRs, fragments of this k-step and the next in VGPRs.
// Up to 128 rows it is a weight stream: (stages - 1) x column blocks x 4 KB of weights in flight a CU, 40 to 96 KB, in a ring that takes
// most of the LDS.
// The operands change places (D^T = W A^T): a lane then holds four consecutive columns of one row.
// Sums run over K in the order of the kernel for row-major weights and with the same rounding: results are equal bit for bit for
// equal splits, whatever the tile.
// MI355X, weights rotating, against the kernels with 32x32x16 before it, as many parts up to 128 rows and no fewer above.  Above 128 rows
// (5 x 2 and 4 x 2 row and column tiles of 32 a wave, loads by four waves of their own; 256 x 256 and 192 x 320 for gate/up):
// 320 x 28672 x 4096 82 -> 70 us, 512 x 28672 x 4096 107 -> 94, 1317 x 28672 x 4096 273 -> 256, 320 x 6144 x 4096 27.4 -> 24.3, 512 x 6144
// x 4096 34.0 -> 30.3, 320 x 4096 x 4096 23.3 -> 20.2, 320 x 4096 x 14336 41.3 -> 40.6, 1317 x 4096 x 14336 174 -> 126, 1632 x 6144 x
// 4096 121 -> 75; 1344 x 128256 x 4096 with arg-max 1190 -> 1010.  Up to 128 rows (weights in register rings): 68 x 28672 x 4096 43.9 ->
// 41.4, 101 x 28672 x 4096 50.5 -> 47.0, 68 x 6144 x 4096 14.0 -> 12.1, 68 x 4096 x 4096 11.3 -> 9.7, 68 x 4096 x 14336 25.3 -> 21.6,
// 101 x 6144 x 4096 16.3 -> 14.4, one row x 6144 x 4096 10.2 -> 9.5; 68 x 128256 x 4096 with arg-max 204 -> 166; not 101 x 4096 x 4096,
// 12.2 -> 13.5, and x 14336, 26.6 -> 28.1.
#pragma once
#include <algorithm>
#include <type_traits>
#include <utility>

#include "esp_gemm_common.h"

namespace {

// A tile of 32 RT x 32 CT, a wave with a 16-row half of every row tile and a 16-column half of every block of 32 columns.  Stages
// in LDS: whole chunks of both operands, STAGES of them (W_HALVES 0: what three times fits, one barrier a chunk), or STAGES + 1
// chunks of activations and W_HALVES half chunks of weights (one barrier a half chunk; up to 160 KB that way).
template <int RT_, int CT_, int STAGES_, int W_HALVES_>
struct GemmTile {
  static constexpr int RT = RT_, CT = CT_;
  static constexpr bool WHOLE = W_HALVES_ == 0;
  static constexpr int S = STAGES_;
  static constexpr int DA = WHOLE ? S - 1 : S, DW = W_HALVES_;          // how far ahead: chunks of activations, half chunks of weights
  static constexpr int ROWS = 32 * RT;
  static constexpr int A_STAGE = RT * 4096, W_STAGE = WHOLE ? CT * 4096 : CT * 2048, A_STAGES = WHOLE ? S : DA + 1, W_STAGES = WHOLE ? S : DW;
  // Loads of a wave.  Half chunks: step j issues the weights of j + DW, then part (j + 1) % 2 of the activations of chunk
  // (j + 1) / 2 + DA.  Whole chunks: as items, pairs of weight pieces first; the first ITEMS0 of chunk c + S go out in c's second
  // step, the others in the step after it.
  static constexpr int W_LOADS = CT / 2, A_LOADS0 = (RT + 1) / 2, A_LOADS1 = RT - A_LOADS0;
  static constexpr int W_ITEMS = WHOLE ? CT / 2 : (CT + 2) / 4, ITEMS = CT / 2 + RT, ITEMS0 = (ITEMS + 1) / 2;
  static constexpr int ACT_LD = CT * 32 + 16;                          // bytes of a SwiGLU result row in LDS
  static constexpr size_t LDS = (size_t)A_STAGES * A_STAGE + (size_t)W_STAGES * W_STAGE;
  static constexpr int TAIL = WHOLE ? S : DA + 1 > (DW + 1) / 2 ? DA + 1 : (DW + 1) / 2;   // chunks whose steps are code of their own
  static_assert(RT * CT <= 64, "accumulators fill the AGPRs");
  static_assert(CT % 2 == 0 && LDS <= 160 * 1024 && (size_t)ROWS * ACT_LD <= LDS, "fits the CU");
  static_assert(WHOLE ? S >= 3 : DW <= 2 * DA + 2 && DW >= 2 * DA - 3, "the loads that a step waits past are all issued by then");
  // loads of a step with e half chunks left, its own among them (even: the first half of a chunk); half chunks
  static constexpr int w_issued(int e) { return e > DW ? W_LOADS : 0; }
  static constexpr int a_issued(int e) { return e > 2 * DA + 1 ? (e % 2 == 0 ? A_LOADS1 : A_LOADS0) : 0; }
  // Loads retire in order: how many younger ones may be in flight at the start of that step.  It reads the weights of the
  // next half chunk and, in a chunk's second half, the next chunk's activations.
  static constexpr int wait(int e) {
    if (WHOLE) {                                         // chunk c + 1 has landed, what there is of c + 2 .. c + S - 1 has not
      const int left = (e + 1) / 2 - 2;
      return (left < S - 2 ? left : S - 2) * (CT + RT);
    }
    int n = a_issued(e + DW - 1);
    for (int x = e + DW - 2; x > e; --x) n += w_issued(x) + a_issued(x);
    if (e % 2 == 1) {
      int na = 0;
      for (int x = e + 2 * DA - 2; x > e; --x) na += w_issued(x) + a_issued(x);
      n = na < n ? na : n;
    }
    return n;
  }
  static constexpr int first_wait() {                    // before the first step: half chunk 0 has landed
    if (WHOLE) return (S - 2) * (CT + RT) + (ITEMS0 < W_ITEMS ? 2 * ITEMS0 : W_ITEMS + ITEMS0);
    int n = 0;
    const int jj = DW < 2 * DA ? DW : 2 * DA;
    for (int j = jj - 1; j >= 1; --j) n += W_LOADS + a_issued(1000 + j);
    if (DW < 2 * DA) n += a_issued(1000 + DW);
    return n;
  }
};

// Order of a k-step's MFMAs: 2 x 2 tiles at a time, so that each shares an operand with the one before (2.01 -> 2.07 PFLOP/s
// from registers), and of the reads of its fragments: as they are needed.
template <int RT, int CT>
struct MfmaOrder {
  int row[RT * CT], col[RT * CT], read[RT + CT];
  constexpr MfmaOrder() : row(), col(), read() {
    int n = 0;
    bool fwd = true;
    for (int p = 0; p < RT; p += 2) {
      const bool two = p + 1 < RT;
      int r = 0;
      for (int k = 0; k < CT; k += 2) {
        const int c0 = fwd ? k : CT - 1 - k, c1 = fwd ? k + 1 : CT - 2 - k;
        row[n] = p + r; col[n++] = c0;
        row[n] = p + r; col[n++] = c1;
        if (two) {
          r ^= 1;
          row[n] = p + r; col[n++] = c1;
          row[n] = p + r; col[n++] = c0;
        }
      }
      fwd = !fwd;
    }
    bool seen[RT + CT] = {};
    int m = 0;
    for (int i = 0; i < RT * CT; ++i) {
      if (!seen[row[i]]) { seen[row[i]] = true; read[m++] = row[i]; }
      if (!seen[RT + col[i]]) { seen[RT + col[i]] = true; read[m++] = RT + col[i]; }
    }
  }
};

// One 16-byte piece per lane, or two that are 1 KB apart in memory and in LDS, global -> LDS (load_to_lds16_sbase; without putting
// M0 back, which costs the one wave of a SIMD two issue slots a load: M0 is named as changed).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <bool NT>
__device__ __forceinline__ void lds_load16(const void* sbase, uint32_t lane_off, uint32_t lds_addr) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds_addr), "v"(lane_off), "s"(sbase) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(lane_off), "s"(sbase) : "memory", "m0");
}
template <bool NT, int OFF = 0>
__device__ __forceinline__ void lds_load16x2(const void* sbase, uint32_t lane_off, uint32_t lds_addr) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3 nt\n\tglobal_load_lds_dwordx4 %1, %2 offset:%4 nt"
                 ::"s"(lds_addr), "v"(lane_off), "s"(sbase), "n"(OFF), "n"(OFF + 1024) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3\n\tglobal_load_lds_dwordx4 %1, %2 offset:%4"
                 ::"s"(lds_addr), "v"(lane_off), "s"(sbase), "n"(OFF), "n"(OFF + 1024) : "memory", "m0");
}
#pragma clang diagnostic pop

template <int... t, typename F>
__device__ __forceinline__ void for_each_const(std::integer_sequence<int, t...>, F f) {
  (f(std::integral_constant<int, t>{}), ...);
}

// EPI: 0 fp32 tile out; 1 per-row arg-max over the workgroup's columns (pairs (value, column) to `pairs`, [n_tiles][M]); 2 SwiGLU of
// column blocks that alternate between gate and up, bf16 [M][N / 2] to out; 3 both 0 and 1.  1 to 3 need splits == 1.
// NT_W: weights by nontemporal loads.  m_live (may be null): how many of the M rows are there (packed rows of a ragged batch); the
// grid was sized for M, the tiles that are there take its first workgroups, strides stay those of M, and every row of the last
// tile that is not there is loaded from the first of them, in which the forward pass keeps zeros (launch_embed).
template <class T, int EPI, bool NT_W>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_gemm_tile(
    const bf16_t* __restrict__ A, const int32_t* __restrict__ a_rows, const bf16_t* __restrict__ W, float* __restrict__ out,
    int M, int N, int K, int splits, int m_tiles, int n_tiles, const int32_t* __restrict__ draw_pos, uint32_t seed,
    const int32_t* __restrict__ m_live, float* __restrict__ pairs) {
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int RT = T::RT, CT = T::CT, DA = T::DA, DW = T::DW;
  n_tiles = with_args(n_tiles, A, a_rows, W, M, N, K, splits, m_tiles);
  const int M_ld = M;
  if (m_live) {                                          // only the first *m_live rows are there
    M = min(*m_live, M);
    if (M <= 0) return;
    m_tiles = (M + T::ROWS - 1) / T::ROWS;
  }
  const int m_last = m_live ? min(M, M_ld - 1) : M - 1;
  const int total = m_tiles * n_tiles * splits;
  const int per_xcd = (total + 7) >> 3;
  if ((int)(blockIdx.x >> 3) >= per_xcd) return;
  const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (logical >= total) return;
  const unsigned ti = (unsigned)logical / (unsigned)m_tiles;
  const int mi = logical - (int)ti * m_tiles, z = (int)(ti / (unsigned)n_tiles), ni = (int)ti - z * n_tiles;
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  const int mt0 = mi * T::ROWS;
  const int blk0 = ni * CT, nblk = N >> 5;
  const int chunks = K / KC, cps = (int)((unsigned)(chunks + splits - 1) / (unsigned)splits), c_begin = z * cps;
  const int nc = min(chunks, c_begin + cps) - c_begin;

  f32x4_t acc[RT][CT];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;
  if (nc > 0) {
    constexpr MfmaOrder<RT, CT> ORDER{};
    // row r of 128 bytes keeps its eight 16-byte pieces XOR-swizzled, so that the fragment reads below are free of bank conflicts
    auto swz = [](int r) { return (r >> 1) & 3; };
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds, ldsw = lds0 + T::A_STAGES * T::A_STAGE;
    const int a_row0 = a_rows ? 0 : mt0;                 // lane offsets have 32 bits: from the tile's first row, or over all rows of a list
    uint32_t aoff[RT];                                   // this lane's piece of row tile j: row 8 wave + lane / 8 of 32
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      const int rt = 8 * wave + (lane >> 3);
      int m = min(mt0 + j * 32 + rt, m_last);
      if (a_rows) m = max(a_rows[m], 0);
      aoff[j] = (uint32_t)(((size_t)(m - a_row0) * K + 8 * ((lane & 7) ^ swz(rt))) * 2);
    }
    const unsigned char* a_base = reinterpret_cast<const unsigned char*>(A) + ((size_t)a_row0 * K + (size_t)c_begin * KC) * 2;
    const size_t W_CHUNK = (size_t)nblk * 4096;
    const uint32_t lane16 = (uint32_t)lane * 16;
    auto load_a = [&](int j, int c, uint32_t stage) { lds_load16<false>(a_base + (size_t)c * (KC * 2), aoff[j], lds0 + stage + (wave + 4 * j) * 1024); };
    // weights: blocks wave, wave + 4, ...; two left over are shared by the four waves
    constexpr int RUNS = (CT + 2) / 4;
    const unsigned char* w_src[RUNS];
    uint32_t w_dst[RUNS];
    constexpr int BLK = T::WHOLE ? 4096 : 2048;           // bytes of a block in a stage
#pragma unroll
    for (int j = 0; j < RUNS; ++j) {
      const bool shared = CT % 4 == 2 && j == RUNS - 1;
      const int b = shared ? 4 * j + (wave >> 1) : wave + 4 * j, off = shared ? (wave & 1) * (BLK / 2) : 0;
      w_src[j] = reinterpret_cast<const unsigned char*>(W) + (size_t)c_begin * W_CHUNK + (size_t)min(blk0 + b, nblk - 1) * 4096 + off;
      w_dst[j] = ldsw + b * BLK + off;
    }
    // item q of a stage of weights: a pair of pieces, or one where a half chunk's block is shared
    auto load_w = [&](int q, int h, uint32_t stage) {
      if constexpr (T::WHOLE) {
        const unsigned char* src = w_src[q >> 1] + (size_t)h * W_CHUNK;   // h: chunk
        if (q & 1) lds_load16x2<NT_W, 2048>(src, lane16, w_dst[q >> 1] + stage);
        else lds_load16x2<NT_W, 0>(src, lane16, w_dst[q >> 1] + stage);
      } else {
        const unsigned char* src = w_src[q] + (size_t)(h >> 1) * W_CHUNK + (h & 1) * 2048;
        if (CT % 4 == 2 && q == RUNS - 1) lds_load16<NT_W>(src, lane16, w_dst[q] + stage);
        else lds_load16x2<NT_W>(src, lane16, w_dst[q] + stage);
      }
    };
    auto load_item = [&](int q, int c, uint32_t astage, uint32_t wstage) {
      if (q < T::W_ITEMS) load_w(q, c, wstage);
      else load_a(q - T::W_ITEMS, c, astage);
    };
    // Lane (r, q) of a fragment holds row r, 16-byte piece 4 (q & 1) + 2 ks + q / 2 of the chunk (k-step ks of two): the pieces
    // in the order in which the 16-wide steps of the kernel for row-major weights take them.
    int a_rd[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) a_rd[ks] = (wm * 16 + lr) * 128 + (((4 * (lq & 1) + 2 * ks + (lq >> 1)) ^ swz(lr)) << 4);
    const int w_rd = T::A_STAGES * T::A_STAGE + (lq >> 1) * 1024 + (lq & 1) * 512 + wn * 256 + lr * 16;
    bf16x8_t af[2][RT], wf[2][CT];
    auto read_frag = [&](int buf, uint32_t astage, uint32_t wstage, int ks, int f) {
      if (f < RT) af[buf][f] = *reinterpret_cast<const bf16x8_t*>(lds + astage + f * 4096 + a_rd[ks]);
      else wf[buf][f - RT] = *reinterpret_cast<const bf16x8_t*>(lds + wstage + (f - RT) * BLK + w_rd + (T::WHOLE ? ks * 2048 : 0));
    };
    // Before the first step: what the steps before it would have loaded (chunks past the end: the last one again, into
    // stages that nobody reads).
    if constexpr (T::WHOLE) {
#pragma unroll
      for (int ch = 0; ch < T::S - 1; ++ch)
#pragma unroll
        for (int q = 0; q < T::ITEMS; ++q) load_item(q, min(ch, nc - 1), ch * T::A_STAGE, ch * T::W_STAGE);
#pragma unroll
      for (int q = 0; q < T::ITEMS0; ++q) load_item(q, min(T::S - 1, nc - 1), (T::S - 1) * T::A_STAGE, (T::S - 1) * T::W_STAGE);
    } else {
      constexpr int PRE = DW > 2 * DA + 1 ? DW : 2 * DA + 1;
#pragma unroll
      for (int j = -PRE; j < 0; ++j) {
        if (j + DW >= 0) {
#pragma unroll
          for (int l = 0; l < T::W_ITEMS; ++l) load_w(l, min(j + DW, 2 * nc - 1), (uint32_t)(j + DW) * T::W_STAGE);
        }
        const int idx = j + 1 + 2 * DA;
        if (idx >= 0) {
#pragma unroll
          for (int l = 0; l < RT; ++l)
            if ((l < T::A_LOADS0) == ((idx & 1) == 0)) load_a(l, min(idx >> 1, nc - 1), (uint32_t)(idx >> 1) * T::A_STAGE);
        }
      }
    }
    wait_loads_but<T::first_wait()>();
    __syncthreads();
#pragma unroll
    for (int f = 0; f < RT + CT; ++f) read_frag(0, 0, 0, 0, f);
    uint32_t a_prev = DA * T::A_STAGE, a_cur = 0, a_next = T::A_STAGE, w_prev = (T::W_STAGES - 1) * T::W_STAGE, w_cur = 0, w_next = T::W_STAGE;
    int c = 0;
    constexpr int SLOTS = RT * CT, READS = RT + CT;
    // One half chunk: the MFMAs of its k-step, and in their shadow the fragments of the next one and the loads of later ones.
    // The barrier at its start says that what those reads need has landed and that every wave has read what the loads overwrite.
    // E: half chunks left, this one among them (1000 and 1001: more than the loads reach ahead).
    auto step = [&](auto e_const) {
      constexpr int E = decltype(e_const)::value, HF = E & 1;
      constexpr bool MORE = E > 1;
      // items of this step's loads: [0, NW) weights and NA activations from A0 on; WHOLE: [Q0, Q0 + NI) of a chunk
      constexpr int NW = T::w_issued(E) ? T::W_ITEMS : 0, NA = T::a_issued(E), A0 = HF ? 0 : T::A_LOADS0;
      constexpr int Q0 = HF ? 0 : T::ITEMS0, NQ = (HF ? E > 2 * T::S - 1 : E > 2 * T::S - 2) ? (HF ? T::ITEMS0 : T::ITEMS - T::ITEMS0) : 0;
      constexpr int NI = T::WHOLE ? NQ : NW + NA;
      if constexpr (MORE && (HF || !T::WHOLE)) {
        wait_loads_but<T::wait(E)>();
        __syncthreads();
      }
#pragma unroll
      for (int k = 0; k < SLOTS; ++k) {
        if (MORE) {
#pragma unroll
          for (int q = 0; q < READS; ++q)
            if (q * (SLOTS * 3 / 4) / READS == k) read_frag(HF ^ 1, HF ? a_next : a_cur, T::WHOLE && !HF ? w_cur : w_next, HF ^ 1, ORDER.read[q]);
        }
        if constexpr (NI > 0) {
#pragma unroll
          for (int q = 0; q < NI; ++q)
            if ((2 * q + 1) * SLOTS / (2 * NI) == k) {
              if constexpr (T::WHOLE) load_item(Q0 + q, c + (HF ? T::S : T::S - 1), HF ? a_cur : a_prev, HF ? w_cur : w_prev);
              else if (q < NW) load_w(q, 2 * c + HF + DW, w_cur);
              else load_a(A0 + q - NW, c + HF + DA, HF ? a_cur : a_prev);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        const int i = ORDER.row[k], j = ORDER.col[k];
        // (text: the accumulator stays where it is; left to choose, the compiler moves accumulators between the steps, 3.4
        // times the loop's time at 256 x 256)
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(wf[HF][j]), "v"(af[HF][i]));
        __builtin_amdgcn_sched_barrier(0);
      }
      if (HF || !T::WHOLE) {
        w_prev = w_cur; w_cur = w_next;
        w_next = w_next + T::W_STAGE == (uint32_t)(T::W_STAGES * T::W_STAGE) ? 0u : w_next + T::W_STAGE;
      }
      if (HF) {
        a_prev = a_cur; a_cur = a_next;
        a_next = a_next + T::A_STAGE == (uint32_t)(T::A_STAGES * T::A_STAGE) ? 0u : a_next + T::A_STAGE;
        ++c;
      }
    };
    while (c < nc - T::TAIL) {
      step(std::integral_constant<int, 1000>{});
      step(std::integral_constant<int, 1001>{});
    }
    for_each_const(std::make_integer_sequence<int, T::TAIL>{}, [&](auto t) {
      constexpr int LEFT = T::TAIL - decltype(t)::value;
      if (nc >= LEFT) {
        step(std::integral_constant<int, 2 * LEFT>{});
        step(std::integral_constant<int, 2 * LEFT - 1>{});
      }
    });
    wait_loads_but<0>();
    __syncthreads();                                     // the LDS is free
    asm volatile("s_nop 15\n\ts_nop 15");                // the last MFMAs' results, of which the compiler does not know
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j) asm volatile("" : "+a"(acc[i][j]));
  }
  // a lane holds rows i * 32 + wm * 16 + lr and columns j * 32 + wn * 16 + 4 lq .. + 3
  if constexpr (EPI == 0 || EPI == 3) {
    float* o = out + (size_t)z * M_ld * N;
    const bool vec = ((uintptr_t)out & 15) == 0;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int m = mt0 + i * 32 + wm * 16 + lr;
      if (m < M) {
#pragma unroll
        for (int j = 0; j < CT; ++j) {
          if (blk0 + j < nblk) {
            float* p = o + (size_t)m * N + (blk0 + j) * 32 + wn * 16 + 4 * lq;
            if (vec) *reinterpret_cast<f32x4_t*>(p) = acc[i][j];
            else {
#pragma unroll
              for (int v = 0; v < 4; ++v) p[v] = acc[i][j][v];
            }
          }
        }
      }
    }
  }
  if constexpr (EPI == 1 || EPI == 3) {
    float* red = reinterpret_cast<float*>(lds);          // [2 wave columns][ROWS][2]
    auto scan = [&](auto sampled) {
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        const int rl = i * 32 + wm * 16 + lr;
        const uint32_t pos = sampled ? (uint32_t)draw_pos[min(mt0 + rl, M - 1)] : 0u;
        float best = -INFINITY;
        int bi = 0x7fffffff;
#pragma unroll
        for (int j = 0; j < CT; ++j)
          if (blk0 + j < nblk) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {                // columns ascend: ties keep the lower one
              const int n = (blk0 + j) * 32 + wn * 16 + 4 * lq + v;
              float x = acc[i][j][v];
              if (sampled) x += gumbel_noise(seed, pos, (uint32_t)n);
              if (x > best) { best = x; bi = n; }
            }
          }
#pragma unroll
        for (int o = 32; o >= 16; o >>= 1) {
          const float ov = __shfl_xor(best, o, 64);
          const int oi = __shfl_xor(bi, o, 64);
          if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
        }
        if (lq == 0) { red[(wn * T::ROWS + rl) * 2] = best; red[(wn * T::ROWS + rl) * 2 + 1] = __int_as_float(bi); }
      }
    };
    // (a loop each: with the noise of 256 values a lane as a branch in one, 256 jumps over code that does not fit the instruction cache)
    if (draw_pos) scan(std::true_type{});
    else scan(std::false_type{});
    __syncthreads();
    for (int rl = tid; rl < T::ROWS; rl += 256) {
      float best = red[rl * 2];
      int bi = __float_as_int(red[rl * 2 + 1]);
      const float ov = red[(T::ROWS + rl) * 2];
      const int oi = __float_as_int(red[(T::ROWS + rl) * 2 + 1]);
      if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
      const int m = mt0 + rl;
      if (m < M) {
        pairs[((size_t)ni * M_ld + m) * 2] = best;
        pairs[((size_t)ni * M_ld + m) * 2 + 1] = __int_as_float(bi);
      }
    }
  }
  if constexpr (EPI == 2) {
    bf16_t* act = reinterpret_cast<bf16_t*>(out);
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int p = 0; p < CT / 2; ++p) {
        bf16x4_t x;
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = (bf16_t)silu_mul(acc[i][2 * p][v], acc[i][2 * p + 1][v]);
        *reinterpret_cast<bf16x4_t*>(lds + (size_t)(i * 32 + wm * 16 + lr) * T::ACT_LD + p * 64 + wn * 32 + lq * 8) = x;
      }
    __syncthreads();
    const int ff = N >> 1;
    constexpr int PER_ROW = CT * 2;                      // 16-byte pieces of a row, four to a pair of blocks
    const bool vec = ((uintptr_t)act & 15) == 0;
    for (int e = tid; e < T::ROWS * PER_ROW; e += 256) {
      const int rl = e / PER_ROW, piece = e % PER_ROW, m = mt0 + rl;
      if (m >= M || blk0 + (piece >> 2) * 2 >= nblk) continue;
      const unsigned char* src = lds + (size_t)rl * T::ACT_LD + piece * 16;
      bf16_t* dst = act + (size_t)m * ff + (blk0 >> 1) * 32 + piece * 8;
      if (vec) *reinterpret_cast<u32x4_t*>(dst) = *reinterpret_cast<const u32x4_t*>(src);
      else {
#pragma unroll
        for (int v = 0; v < 8; ++v) dst[v] = reinterpret_cast<const bf16_t*>(src)[v];
      }
    }
  }
}

// The tiles there are, with their index in GEMM_TILES: those for up to 128 rows (weights always by nontemporal loads) and the others.
#define ESP_ROW_TILES(X) X(0, 1, 2, 8, 0) X(1, 1, 4, 6, 0) X(2, 1, 6, 5, 0) X(3, 2, 2, 8, 0) X(4, 2, 4, 4, 0) X(5, 2, 6, 5, 0) X(6, 3, 2, 8, 0) \
  X(7, 3, 4, 4, 0) X(8, 3, 6, 4, 0) X(9, 4, 2, 6, 0) X(10, 4, 4, 5, 0) X(11, 4, 6, 4, 0)
#define ESP_WIDE_TILES(X) X(12, 3, 8, 3, 0) X(13, 4, 4, 5, 0) X(14, 4, 6, 4, 0) X(15, 4, 8, 3, 0) X(16, 5, 6, 3, 0) X(17, 5, 8, 3, 0) \
  X(18, 6, 6, 3, 0) X(19, 6, 8, 2, 5) X(20, 6, 10, 2, 4) X(21, 8, 6, 2, 5) X(22, 8, 8, 2, 4)

// dynamic LDS above the default needs an attribute, set once per kernel
template <class T, int EPI, bool NT>
hipError_t tile_allow_lds() {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(k_gemm_tile<T, EPI, NT>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)T::LDS);
  return attr;
}

template <int EPI>
hipError_t tile_prepare() {
  hipError_t e = hipSuccess;
#define ESP_X(I_, RT_, CT_, S_, H_)                                                 \
  static_assert(GEMM_TILES[I_].rt == RT_ && GEMM_TILES[I_].ct == CT_, "one table"); \
  if (e == hipSuccess) e = tile_allow_lds<GemmTile<RT_, CT_, S_, H_>, EPI, true>();
  ESP_ROW_TILES(ESP_X)
  if constexpr (EPI != 3) { ESP_WIDE_TILES(ESP_X) }
#undef ESP_X
#define ESP_X(I_, RT_, CT_, S_, H_) \
  if (e == hipSuccess) e = tile_allow_lds<GemmTile<RT_, CT_, S_, H_>, EPI, false>();
  if constexpr (EPI != 3) { ESP_WIDE_TILES(ESP_X) }
#undef ESP_X
  return e;
}

template <class T, int EPI, bool NT>
hipError_t tile_launch(hipStream_t st, const TileGemm& g) {
  const hipError_t attr = tile_allow_lds<T, EPI, NT>();
  if (attr != hipSuccess) return attr;
  const int m_tiles = (g.M + T::ROWS - 1) / T::ROWS, n_tiles = ((g.N >> 5) + T::CT - 1) / T::CT;
  const int64_t total = (int64_t)m_tiles * n_tiles * g.splits;
  if (total > INT32_MAX - 8 || !gemm_rows_fit(std::min(g.M, T::ROWS), g.K)) return hipErrorInvalidValue;
  launch_kernel(k_gemm_tile<T, EPI, NT>, dim3((unsigned)((total + 7) / 8 * 8)), dim3(256), T::LDS, st, (const bf16_t*)g.A, g.a_rows,
                (const bf16_t*)g.W, (float*)g.out, g.M, g.N, g.K, g.splits, m_tiles, n_tiles, g.draw_pos, g.seed, g.m_live, g.pairs);
  return hipGetLastError();
}

// Weights by nontemporal loads up to 2400 rows.  Eight layers on 2048 keys of the 8B shape, without and with: one row 822 -> 766 us, 30 rows
// 874 -> 829, 68 rows 966 -> 949, 128 rows 1158 -> 1154, 160 rows 1365 -> 1349, 320 rows 1759 -> 1712, 512 rows 2208 -> 2175, batches of 672
// rows 3008 -> 2945, 768 rows 3115 -> 3084, 960 (720 there) 3399 -> 3366, 1344 rows 5039 -> 4983, 2112 rows 7182 -> 7132; four of 1024 keys, 2560
// rows 8.00 -> 8.00 ms, 3200 10.20 -> 10.24, 5120 15.96 -> 16.05 (3584 there 12.40 -> 12.55).
template <int EPI>
hipError_t tile_dispatch(hipStream_t st, const TileGemm& g) {
  [[maybe_unused]] const bool nt = g.M <= 2400;
#define ESP_X(I_, RT_, CT_, S_, H_) \
  case I_: return tile_launch<GemmTile<RT_, CT_, S_, H_>, EPI, true>(st, g);
  switch (g.tile) { ESP_ROW_TILES(ESP_X) }
#undef ESP_X
#define ESP_X(I_, RT_, CT_, S_, H_) \
  case I_: return nt ? tile_launch<GemmTile<RT_, CT_, S_, H_>, EPI, true>(st, g) : tile_launch<GemmTile<RT_, CT_, S_, H_>, EPI, false>(st, g);
  if constexpr (EPI != 3)
    switch (g.tile) { ESP_WIDE_TILES(ESP_X) }
#undef ESP_X
  return hipErrorInvalidValue;
}

}  // namespace
