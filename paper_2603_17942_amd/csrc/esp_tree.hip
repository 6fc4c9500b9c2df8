// Tree logic kept on the device: block descriptor from parent pointers, greedy acceptance + KV
// commit, row lists for the proposal pass, pruning + dynamic tree construction
// (paper Sec. 2 Eq. 3, Sec. 3.3-3.5, Alg. 1, App. C, App. E).  One workgroup per sequence;
// everything is integer work except the fp32 products of Alg. 1.
#include <climits>

#include "esp_internal.h"

namespace {

constexpr int MAXC = 4096;   // candidates Alg. 1 may create (root included)

__device__ __forceinline__ bool kv_seq_ok(const KvDev& kv, int seq, int n_rows, int rows_per_seq) {
  int L = kv.len[seq];
  int base = kv.base[seq];
  int cap = kv.seq_cap[seq];
  return L >= 0 && L <= kv.len_bound && n_rows >= 0 && n_rows <= rows_per_seq && L + n_rows <= cap &&
         base >= 0 && (base & 63) == 0 && (int64_t)base + cap <= kv.capacity;
}

__device__ __forceinline__ int lanes_below(unsigned long long ballot) {   // set bits below this lane
  return __builtin_amdgcn_mbcnt_hi((unsigned)(ballot >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)ballot, 0u));
}

// Writes every derived per-row array of one sequence.  Called by all threads of the workgroup with the
// structure of the node rows in LDS: node_parent(i), node_depth(i), node_anc(i, w) = word w of the bitset
// of i and its ancestors (w < node_words).  Rows go out in row order, whole lines at a time; nothing that
// was written is read back.  A tree that does not fit the block sets the status word instead.
template <typename Parent, typename Depth, typename Anc>
__device__ void write_rows(int seq, int rows_per_seq, int k, int layout, int anc_words, int n_nodes, int node_words,
                           Parent node_parent, Depth node_depth, Anc node_anc, int32_t* n_rows, int32_t* tok,
                           int32_t* parent, int32_t* depth, int32_t* mask_j, int32_t* attach, uint64_t* anc,
                           int32_t* status) {
  const size_t r0 = (size_t)seq * rows_per_seq;
  const int owners = k == 0 ? 0 : (layout == ESP_LAYOUT_PER_NODE ? n_nodes : 1);
  const int total = n_nodes + owners * k;
  if (n_nodes < 1 || total > rows_per_seq || (total + 63) / 64 > anc_words) {
    if (threadIdx.x == 0) { atomicOr(status, ESP_DEV_BAD_TREE); n_rows[seq] = 0; }
    return;
  }
  // mask rows: chain j = 1..k of owner a sits at n_nodes + a*k + (j-1)
  for (int row = threadIdx.x; row < total; row += blockDim.x) {
    const int t = row - n_nodes;
    const int a = t < 0 ? row : t / k, j = t < 0 ? 0 : t - a * k + 1;
    depth[r0 + row] = node_depth(a) + j;
    mask_j[r0 + row] = j;
    attach[r0 + row] = a;
    parent[r0 + row] = j == 0 ? node_parent(row) : (j == 1 ? a : row - 1);
    if (j > 0) tok[r0 + row] = -1;
  }
  for (int i = threadIdx.x; i < total * anc_words; i += blockDim.x) {
    const int row = i / anc_words, w = i - row * anc_words;
    const int t = row - n_nodes;
    const int a = t < 0 ? row : t / k;
    uint64_t bits = w < node_words ? node_anc(a, w) : 0ull;
    if (t >= 0) {                                       // plus the rows of its own chain up to itself
      const int lo = max(n_nodes + a * k, w * 64), hi = min(row, w * 64 + 63);
      if (lo <= hi) bits |= (~0ull >> (63 - (hi - lo))) << (lo & 63);
    }
    anc[r0 * anc_words + i] = bits;
  }
  if (threadIdx.x == 0) n_rows[seq] = total;
}

// Block descriptor from parent pointers.  Trees here can be a prompt's chain of up to 1024 nodes, so
// nothing walks parent by parent: a wave takes 64 consecutive nodes and closes the ancestor sets inside
// them by pointer jumping (six rounds of lane exchanges); what lies before those 64 nodes is the finished
// set of the first ancestor outside, copied word by word, one 64-node group after the other.
// 512-node chain: 12 us (250 us walking one pointer at a time through global memory).
constexpr int FROM_TREE_LDS_PER_NODE = 24;   // ancestor mask inside the group, outside ancestor, depth, parent

__global__ __launch_bounds__(256) void k_block_from_tree(int rows_per_seq, int k, int layout, int anc_words,
                                                         int32_t* n_rows, const int32_t* n_nodes_arr, int32_t* tok,
                                                         int32_t* parent, int32_t* depth, int32_t* mask_j,
                                                         int32_t* attach, uint64_t* anc, int32_t* status) {
  extern __shared__ __align__(16) unsigned char raw[];
  const int seq = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = n_nodes_arr[seq];
  const size_t r0 = (size_t)seq * rows_per_seq;
  const int nw = (min(max(n, 0), rows_per_seq) + 63) >> 6;             // groups = words of a node's set
  uint64_t* s_anc = reinterpret_cast<uint64_t*>(raw);                  // [rows_per_seq][nw]
  uint64_t* s_mask = s_anc + (size_t)rows_per_seq * anc_words;         // [rows_per_seq]
  int32_t* s_ext = reinterpret_cast<int32_t*>(s_mask + rows_per_seq);
  int32_t* s_dep = s_ext + rows_per_seq;
  int32_t* s_par = s_dep + rows_per_seq;
  bool bad = n < 1 || n > rows_per_seq;
  if (!bad)
    for (int i = tid; i < n; i += blockDim.x) {
      const int p = parent[r0 + i];
      s_par[i] = p;
      if (i == 0 ? p != -1 : (p < 0 || p >= i)) bad = true;
    }
  if (__syncthreads_or(bad)) {
    if (tid == 0) { atomicOr(status, ESP_DEV_BAD_TREE); n_rows[seq] = 0; }
    return;
  }
  for (int g = wave; g < nw; g += 4) {
    const int row = g * 64 + lane;
    const int p = row < n ? s_par[row] : -1;
    int jump = p >= g * 64 ? p - g * 64 : -1, d = jump >= 0 ? 1 : 0, ext = p;
    unsigned long long mask = 1ull << lane;
    while (__builtin_amdgcn_ballot_w64(jump >= 0)) {                    // at most six rounds: the hops double
      const int from = jump >= 0 ? jump : lane;
      const unsigned long long om = __shfl(mask, from, 64);
      const int oj = __shfl(jump, from, 64), od = __shfl(d, from, 64), oe = __shfl(ext, from, 64);
      if (jump >= 0) { mask |= om; d += od; jump = oj; ext = oe; }
    }
    if (row < n) { s_mask[row] = mask; s_ext[row] = ext; s_dep[row] = d; }
  }
  __syncthreads();
  for (int g = 0; g < nw; ++g) {
    const int rows_g = min(64, n - g * 64);
    for (int i = tid; i < 64 * nw; i += blockDim.x) {
      const int row = g * 64 + (i & 63), w = i >> 6;
      if ((i & 63) < rows_g) {
        const int e = s_ext[row];
        s_anc[(size_t)row * nw + w] = w == g ? s_mask[row] : (w < g && e >= 0 ? s_anc[(size_t)e * nw + w] : 0ull);
        if (w == 0 && e >= 0) s_dep[row] += s_dep[e] + 1;
      }
    }
    __syncthreads();
  }
  write_rows(seq, rows_per_seq, k, layout, anc_words, n, nw, [&](int i) { return s_par[i]; },
             [&](int i) { return s_dep[i]; }, [&](int i, int w) { return s_anc[(size_t)i * nw + w]; }, n_rows, tok, parent,
             depth, mask_j, attach, anc, status);
}

// ---- greedy verification (Sec. 2 Eq. 3) -----------------------------------------------------------------
__global__ __launch_bounds__(256) void k_verify(BlockDev b, KvDev kv, const int32_t* __restrict__ g,
                                                int32_t* n_emit, int32_t* emit_tok, int32_t* accepted_row,
                                                int32_t* star_row) {
  __shared__ int s_next;
  const int seq = blockIdx.x;
  const size_t r0 = (size_t)seq * b.rows_per_seq;
  const int nn = b.n_nodes[seq], nr = b.n_rows[seq];
  int32_t* et = emit_tok + (size_t)seq * (ESP_MAX_MASKS + 1);
  int32_t* ar = accepted_row + (size_t)seq * (ESP_MAX_MASKS + 1);
  if (!kv_seq_ok(kv, seq, nr, b.rows_per_seq) || nn < 1 || nn > nr) {
    if (threadIdx.x == 0) { n_emit[seq] = 0; star_row[seq] = 0; }
    return;
  }
  int cur = 0, a = 0;
  if (threadIdx.x == 0) ar[0] = 0;
  while (a < ESP_MAX_MASKS) {
    if (threadIdx.x == 0) s_next = 0x7fffffff;
    __syncthreads();
    const int want = g[r0 + cur];
    for (int c = threadIdx.x; c < nn; c += blockDim.x)
      if (b.parent[r0 + c] == cur && b.tok[r0 + c] == want) atomicMin(&s_next, c);   // first match in row order
    __syncthreads();
    const int nxt = s_next;
    __syncthreads();
    if (nxt == 0x7fffffff) break;
    if (threadIdx.x == 0) { et[a] = b.tok[r0 + nxt]; ar[a + 1] = nxt; }
    cur = nxt;
    ++a;
  }
  if (threadIdx.x == 0) {
    et[a] = g[r0 + cur];
    n_emit[seq] = a + 1;
    star_row[seq] = cur;
    kv.len[seq] += a + 1;
  }
}

// moves the accepted rows' K/V to slots L+1.. in path order; one workgroup per (layer*kv_head, seq),
// one thread per feature, accepted rows processed in order (a destination can be a later source).
template <typename T>
__global__ void k_kv_commit(BlockDev b, KvDev kv, int n_kv, int hd, const int32_t* __restrict__ n_emit,
                            const int32_t* __restrict__ accepted_row) {
  const int seq = blockIdx.y;
  const int ne = n_emit[seq];
  if (ne < 2) return;
  const int layer = blockIdx.x / n_kv, kvh = blockIdx.x % n_kv;
  const int d = threadIdx.x;
  const int L = kv.len[seq] - ne;    // k_verify already advanced len
  const int64_t base = kv.base[seq];
  T* kp = (T*)kv.k + kv_plane(layer, kvh, n_kv, kv.capacity, hd);
  T* vp = (T*)kv.v + kv_plane(layer, kvh, n_kv, kv.capacity, hd);
  const int32_t* ar = accepted_row + (size_t)seq * (ESP_MAX_MASKS + 1);
  for (int i = 1; i < ne; ++i) {
    int64_t src = base + L + ar[i], dst = base + L + i;
    if (src == dst) continue;
    kp[k_off(dst, d, hd)] = kp[k_off(src, d, hd)];
    vp[v_off(dst, d, hd)] = vp[v_off(src, d, hd)];
  }
}

// rows whose logits seed the next tree (Sec. 3.3): mask rows aligned to the accepted position
__global__ void k_mask_rows(BlockDev b, const int32_t* star_row, const int32_t* n_emit, int32_t* a_rows,
                            int32_t* n_lists) {
  const int seq = blockIdx.x;
  const int k = b.k_masks;
  const int nn = b.n_nodes[seq], nr = b.n_rows[seq], ne = n_emit[seq];
  int lists = 0, first = 0;
  if (ne >= 1 && nn >= 1 && nr <= b.rows_per_seq) {
    if (b.layout == ESP_LAYOUT_PER_NODE) {
      int s = star_row[seq];
      if (s >= 0 && s < nn && nn * (k + 1) == nr) { lists = k; first = nn + s * k; }
    } else {
      int a = ne - 1;
      if (nn + k == nr && a < k) { lists = k - a; first = nn + a; }
    }
  }
  for (int i = threadIdx.x; i < k; i += blockDim.x)
    a_rows[seq * k + i] = i < lists ? seq * b.rows_per_seq + first + i : -1;
  if (threadIdx.x == 0) n_lists[seq] = lists;
}

// ---- pruning + dynamic tree (Alg. 1, Sec. 3.5) -----------------------------------------------------------
// Candidates of Alg. 1 that can still be part of the tree.  The tree is the root plus the B - 1 most
// probable of all candidates, a child is never more probable than its parent and is created after it:
// so a candidate that is not among the B - 1 best created so far is out for good, and so is everything
// that would grow from it.  Only the best B - 1 are kept from depth to depth (sorted), and of a depth's
// children only those are created that beat the last of a full set.  Relative creation order, which
// breaks ties and orders rows, is what the creation index records.
// A list entry above 1 (or NaN) voids the second premise: then every candidate is created and stays in the pool
// that the selections choose from, as Alg. 1 is written ("wide" below).
constexpr int MAX_CAND = MAXC + ESP_MAX_TREE_NODES + 4;
struct TreeLds {
  // every candidate created, by creation index (0 = the root)
  int32_t tok[MAXC];
  int16_t par[MAXC];
  uint8_t dep[MAXC];
  uint8_t used[MAXC];           // has been in the node set N
  // the kept candidates, sorted, followed by a depth's new ones: probability and creation index; two
  // buffers, a selection writes the other one
  __align__(16) float prob[2][MAX_CAND];
  int32_t cre[2][MAX_CAND];
  __align__(16) float pick_p[ESP_MAX_TREE_NODES + 4];   // survivors of a selection, in list order
  int32_t pick[ESP_MAX_TREE_NODES];
  int32_t expand[ESP_MAX_TREE_NODES];      // list places of the kept candidates to expand next, in order
  __align__(16) uint32_t order[ESP_MAX_TREE_NODES];   // depth << 16 | creation index of the kept nodes
  int32_t row_tok[ESP_MAX_TREE_NODES], row_par[ESP_MAX_TREE_NODES], row_dep[ESP_MAX_TREE_NODES];
  uint64_t row_anc[ESP_MAX_TREE_NODES][ESP_MAX_TREE_NODES / 64];
  int16_t row_of[MAXC];                    // creation index -> row, -1: not in the tree
  int32_t list_id[ESP_MAX_MASKS * ESP_MAX_TOPK];   // the sequence's Top-K' lists, staged once
  float list_p[ESP_MAX_MASKS * ESP_MAX_TOPK];
  uint64_t count[2][4];                    // pick_best: per-wave counts
  int32_t n_cand, n_keep, kept_buf;        // n_keep -1: more candidates or nodes than there is room for
  int32_t orphan;                          // a kept node whose parent is not
  __align__(16) int32_t odd[4];            // per wave: an entry outside [0, 1] among those it staged
  float all_p[MAXC];                       // wide: probability by creation index
  int32_t n_cre, n_pool;                   // wide: candidates created + 1, candidates not used yet
};

// The whole workgroup, for more candidates than it has threads: the T best (T <= 255) of the n in buffer
// `from`, unsorted but in list order, to s.pick / pick_p.  The T-th largest probability (as a bit pattern) is found
// two bits at a time from the top: each wave counts, over its quarter of the list, the values that reach the three
// prefixes with those bits set (ballot, popcount), and the four waves' counts meet in LDS, one barrier a step.
// Up to PICK_REGS * 256 candidates a step reads no LDS but the counts.  With the ranking below, the build at B = 256,
// k = 3, K = 12: 37 us; 70 us with one wave that counts bit by bit over LDS and ranks by lane reads, 42 us with
// a histogram over all candidates.
constexpr int PICK_REGS = 5;
__device__ void pick_best(TreeLds& s, int from, int n, int T) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int quarter = ((n + 255) >> 8) << 6;               // whole groups of 64
  const int j0 = wave * quarter, j1 = min(n, j0 + quarter);
  const float* v = s.prob[from];
  auto bits_at = [&](int j) {                              // 0 past the quarter's end: never counted
    const uint32_t u = __float_as_uint(v[min(j + lane, n - 1)]);
    return j + lane < j1 ? u : 0u;
  };
  uint32_t held[PICK_REGS];
#pragma unroll
  for (int r = 0; r < PICK_REGS; ++r) held[r] = bits_at(j0 + 64 * r);
  uint32_t bound = 0;
  int reach = n, turn = 0;
#pragma unroll 1
  for (int shift = 30;; shift -= 2, turn ^= 1) {
    // last of all, how many lie above the bound and how many are equal to it
    const bool done = reach == T || shift < 0;
    const uint32_t a = done ? max(bound, 1u) : bound | 1u << shift, b = done ? bound + 1 : bound | 2u << shift,
                   c = done ? ~0u : bound | 3u << shift;
    int na = 0, nb = 0, nc = 0;
    auto count = [&](uint32_t u) {
      na += __popcll(__builtin_amdgcn_ballot_w64(u >= a));
      nb += __popcll(__builtin_amdgcn_ballot_w64(u >= b));
      nc += __popcll(__builtin_amdgcn_ballot_w64(u >= c));
    };
#pragma unroll
    for (int r = 0; r < PICK_REGS; ++r)
      if (64 * r < quarter) count(held[r]);
#pragma unroll 1
    for (int j = j0 + 64 * PICK_REGS; j < j1; j += 64) count(bits_at(j));
    if (lane == 0) s.count[turn][wave] = (uint64_t)na | (uint64_t)nb << 16 | (uint64_t)nc << 32;
    __syncthreads();
    if (done) break;
    const uint64_t all = s.count[turn][0] + s.count[turn][1] + s.count[turn][2] + s.count[turn][3];
    const uint32_t ab = __builtin_amdgcn_readfirstlane((uint32_t)all);
    na = ab & 0xffff, nb = ab >> 16, nc = __builtin_amdgcn_readfirstlane((uint32_t)(all >> 32));
    if (nc >= T) { bound |= 3u << shift; reach = nc; }
    else if (nb >= T) { bound |= 2u << shift; reach = nb; }
    else if (na >= T) { bound |= 1u << shift; reach = na; }
  }
  // of those equal to the bound the first in list order are taken
  if (threadIdx.x < 3) s.pick_p[T + threadIdx.x] = __int_as_float(-1);
  int gt = 0, gt_before = 0, eq_before = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const int g = (int)(s.count[turn][w] >> 16) & 0xffff;
    const int e = (bound ? (int)s.count[turn][w] & 0xffff : max(min(n, (w + 1) * quarter) - w * quarter, 0)) - g;
    gt += g;
    if (w < wave) { gt_before += g; eq_before += e; }
  }
  int room = T - gt - eq_before, base = gt_before + min(eq_before, T - gt);
#pragma unroll 1
  for (int j = j0; j < j1; j += 64) {
    const bool in = j + lane < j1;
    const uint32_t u = bits_at(j);
    const unsigned long long be = __builtin_amdgcn_ballot_w64(in && u == bound);
    const bool sel = in && (u > bound || (u == bound && lanes_below(be) < room));
    room -= __popcll(be);
    const unsigned long long bs = __builtin_amdgcn_ballot_w64(sel);
    const int at = base + lanes_below(bs);
    if (sel) { s.pick[at] = s.cre[from][j + lane]; s.pick_p[at] = __uint_as_float(u); }
    base += __popcll(bs);
  }
}

// The whole workgroup: of the n candidates of buffer `from` the T best (T <= 255), sorted by (probability
// descending, creation ascending), to the other buffer; returns how many.  A thread per candidate
// counts the better ones, four at a time from one LDS read that all lanes share.  Candidates of equal probability
// lie in creation order in both buffers; behind the last one lie three entries worse than anything (-1).
__device__ int keep_best(TreeLds& s, int from, int n, int T) {
  const int tid = threadIdx.x, a0 = tid & ~63;
  const bool pick = n > 256;
  const int m = pick ? T : n;
  if (pick) {
    pick_best(s, from, n, T);
    __syncthreads();
  }
  const float* v = pick ? s.pick_p : s.prob[from];
  const int32_t* c = pick ? s.pick : s.cre[from];
  if (a0 < m) {                                            // wave-uniform
    const int32_t p = tid < m ? __float_as_int(v[tid]) : 0x7fffffff;      // >= 0.0: ordered as integers
    int rank = 0;
    // equal ones before this candidate are better: [0, a0) all lie before it, [a0, a0 + 64) may
    auto better = [&](int b0, int b1, auto before) {
#pragma unroll 2
      for (int b = b0; b < b1; b += 4) {
        const u32x4_t o = *reinterpret_cast<const u32x4_t*>(v + b);
#pragma unroll
        for (int e = 0; e < 4; ++e) rank += (int32_t)o[e] > p - (before(b + e) ? 1 : 0) ? 1 : 0;
      }
    };
    better(0, min(a0, m), [](int) { return true; });
    better(a0, min(a0 + 64, m), [&](int b) { return b < tid; });
    better(a0 + 64, m, [](int) { return false; });
    if (tid < m && rank < T) { s.prob[from ^ 1][rank] = __int_as_float(p); s.cre[from ^ 1][rank] = c[tid]; }
  }
  return min(m, T);
}

// Alg. 1.  One wave creates a depth's candidates and picks the node set (lane exchanges and ballots
// instead of workgroup barriers), the workgroup sorts.  Leaves the kept candidates in
// s.cre[s.kept_buf][0..s.n_keep).  Latency is all there is to it: the code is kept in small loops on
// purpose (it runs once per launch, so instruction fetch costs more than arithmetic).  B = 64, k = 4,
// K = 8: the call takes 14.7 us; 36 us with every candidate created and a histogram per selection.
template <bool wide>
__device__ void grow_tree(TreeLds& s, const esp_tree_params& p, int root_tok, int kp, int depth_limit) {
  const int lane = threadIdx.x & 63;
  const bool first_wave = threadIdx.x < 64;
  const bool is_static = !wide && p.static_widths[0] > 0;
  const int T = max(p.B - 1, 0);
  const int K = p.K, B = p.B, ew = p.expand_width, drop_parent = p.prune_parent, drop_last = p.prune_last;
  // P(child) = P(parent) * P(t|l), one fp32 product (Alg. 1).  Both are >= +0 or a positive NaN, and so is the product
  // (the sign of 0 * infinity is cleared): ordered as integers everywhere
  auto child_prob = [](float parent, float entry) { return wide ? fabsf(parent * entry) : parent * entry; };
  int buf = 0;                      // where the kept candidates are (wide: the node set last chosen)
  int nk = 0;                       // candidates kept (wide: in the pool, which is buffer 0)
  int n_cre = 1;                    // next creation index (first wave)
  int n_exp = 1;                    // nodes to expand: the root first (first wave)
#pragma unroll 1
  for (int i = 1; i <= depth_limit; ++i) {
    if (first_wave) {
      const int want = is_static ? p.static_widths[i - 1] : min(K, B - i);
      const int32_t id = lane < kp ? s.list_id[(i - 1) * kp + lane] : -1;
      const float lp = lane < kp ? s.list_p[(i - 1) * kp + lane] : 0.f;
      const int nv = __builtin_ctzll(__builtin_amdgcn_ballot_w64(id < 0));          // a negative id ends a list
      const int dst = wide ? 0 : buf;
      const int floor_p = !wide && !is_static && T > 0 && nk >= T ? __float_as_int(s.prob[buf][T - 1]) : INT_MIN;
      int n = nk;
#pragma unroll 1
      for (int e0 = 0; e0 < n_exp; e0 += 64) {
        const bool live = e0 + lane < n_exp;
        const int place = live && i > 1 ? s.expand[e0 + lane] : 0;
        const int pcre = i > 1 ? s.cre[buf][place] : 0;
        const int ptok = i > 1 ? s.tok[pcre] : root_tok;
        const float pp = i > 1 ? s.prob[buf][place] : 1.0f;
        // children: the first `want` list entries that survive the pruning rule; created if they can
        // still be part of the tree
        uint32_t make = 0;
        int taken = 0;
#pragma unroll 1
        for (int c = 0, c1 = min(nv, want);; c1 = min(nv, c1 + 1)) {
#pragma unroll 1
          for (; c < c1; ++c) {
            const int t = __builtin_amdgcn_readlane(id, c);
            const float q = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lp), c));
            const bool ok = live && taken < want && !(drop_parent && t == ptok) && !(drop_last && i >= 2 && t == root_tok);
            taken += ok ? 1 : 0;
            if (ok && __float_as_int(child_prob(pp, q)) > floor_p) make |= 1u << c;
          }
          // more entries only where one was dropped
          if (c >= nv || __builtin_amdgcn_ballot_w64(live && taken < want) == 0ull) break;
        }
        const int cnt = __popc(make);
        int off = 0, tot = 0;
#pragma unroll 1
        for (int b = 0; b < 6; ++b) {                     // prefix sum of counts up to 32, bit by bit
          const unsigned long long bb = __builtin_amdgcn_ballot_w64((cnt >> b) & 1);
          off += lanes_below(bb) << b;
          tot += __popcll(bb) << b;
        }
        if (n_cre + tot > MAXC) { n = -1; break; }
#pragma unroll 1
        for (int made = off; make; ++made) {
          const int c = __builtin_ctz(make);
          make &= make - 1;
          const int cre = n_cre + made;
          s.tok[cre] = s.list_id[(i - 1) * kp + c];
          s.par[cre] = (int16_t)pcre;
          s.dep[cre] = (uint8_t)i;
          s.used[cre] = 0;
          s.row_of[cre] = -1;
          const float pc = child_prob(pp, s.list_p[(i - 1) * kp + c]);
          s.prob[dst][n + made] = pc;
          s.cre[dst][n + made] = cre;
          if (wide) s.all_p[cre] = pc;
        }
        n += tot;
        n_cre += tot;
      }
      if (lane < 3 && n >= 0) s.prob[dst][n + lane] = __int_as_float(-1);
      if (lane == 0) { s.n_cand = n; if (wide) s.n_cre = n_cre; }
    }
    __syncthreads();
    int n = s.n_cand;
    if (n < 0) { if (threadIdx.x == 0) s.n_keep = -1; return; }
    if (!wide && n == nk) break;    // nothing new: no deeper node either, and the list is sorted as it is
    const bool last = i == depth_limit || (wide && n == nk);
    if (is_static) {
      // fixed tree: everything is kept, in creation order, and the first fresh child is expanded next
      n_exp = 1;
      if (threadIdx.x == 0) s.expand[0] = nk;
      nk = n;
    } else {
      int src = buf, take = T;
      if (wide) {
        src = 0;
        take = last ? T : max(B - i, 0);
        if (last) {                   // the tree is chosen from all candidates, used ones included
          n = s.n_cre - 1;
          for (int c = threadIdx.x; c < n; c += 256) { s.prob[0][c] = s.all_p[c + 1]; s.cre[0][c] = c + 1; }
          if (threadIdx.x < 3) s.prob[0][n + threadIdx.x] = __int_as_float(-1);
          __syncthreads();
        }
      }
      nk = keep_best(s, src, n, take);
      buf = src ^ 1;
    }
    if (last) break;
    __syncthreads();
    if (first_wave && !is_static) {
      // node set <- the B - i most probable candidates not used before; those of depth i are expanded next
      int room = max(B - i, 0), ne = 0;
      const int width = ew > 0 ? ew : ESP_MAX_TREE_NODES;
#pragma unroll 1
      for (int a0 = 0; a0 < nk; a0 += 64) {
        const int a = a0 + lane;
        const int cre = s.cre[buf][min(a, nk - 1)];
        const bool fresh = a < nk && !s.used[cre];
        const unsigned long long bf = __builtin_amdgcn_ballot_w64(fresh);
        const bool in = fresh && lanes_below(bf) < room;
        room -= __popcll(bf);
        if (in) s.used[cre] = 1;
        const bool ex = in && s.dep[cre] == i;
        const unsigned long long bx = __builtin_amdgcn_ballot_w64(ex);
        const int at = ne + lanes_below(bx);
        if (ex && at < width) s.expand[at] = a;
        ne += __popcll(bx);
      }
      n_exp = min(ne, width);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (wide) {                     // the used ones leave the pool, the others close up
        int left = 0;
#pragma unroll 1
        for (int j = 0; j < n; j += 64) {
          const int at = min(j + lane, n - 1), c = s.cre[0][at];
          const float pc = s.prob[0][at];
          const bool stay = j + lane < n && !s.used[c];
          const unsigned long long bs = __builtin_amdgcn_ballot_w64(stay);
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          if (stay) { s.cre[0][left + lanes_below(bs)] = c; s.prob[0][left + lanes_below(bs)] = pc; }
          left += __popcll(bs);
        }
        if (lane == 0) s.n_pool = left;
      }
    }
    if (wide) {
      __syncthreads();
      nk = s.n_pool;
    }
  }
  if (threadIdx.x == 0) {
    s.n_keep = nk + 1 > ESP_MAX_TREE_NODES ? -1 : nk;
    s.kept_buf = buf;
  }
}

__global__ __launch_bounds__(256) void k_build_tree(esp_tree_params p, const int32_t* __restrict__ topk_id,
                                                    const float* __restrict__ topk_p, int kp,
                                                    const int32_t* __restrict__ n_lists,
                                                    const int32_t* __restrict__ n_emit,
                                                    const int32_t* __restrict__ emit_tok, int rows_per_seq,
                                                    int anc_words, int32_t* n_rows, int32_t* n_nodes, int32_t* tok,
                                                    int32_t* parent, int32_t* depth, int32_t* mask_j,
                                                    int32_t* attach, uint64_t* anc, int32_t* status, int reuse) {
  extern __shared__ __align__(16) unsigned char raw[];
  TreeLds& s = *reinterpret_cast<TreeLds*>(raw);
  const int seq = blockIdx.x, tid = threadIdx.x;
  const size_t r0 = (size_t)seq * rows_per_seq;
  const int ne = n_emit[seq];
  const bool is_static = p.static_widths[0] > 0;
  int depth_limit = min(p.k, n_lists[seq]);
  if (ne < 1 || ne > ESP_MAX_MASKS + 1) {   // sequence skipped upstream
    if (tid == 0) { n_rows[seq] = 0; n_nodes[seq] = 0; atomicOr(status, ESP_DEV_BAD_TREE); }
    return;
  }
  if (is_static && reuse && depth_limit == p.k) {
    // Fixed tree whose rows this block already holds (Sec. 4.3: the descriptor of a static tree is
    // built once): the shape -- root, K_1 children, K_i children under the first node of depth i - 1
    // -- does not depend on the lists, so parents, depths, mask rows and ancestor sets stay and
    // only the tokens are written.  A thread per node walks the chain of first children down to its
    // own depth.  If a list runs out of surviving entries the shape would change: then (all threads
    // agree first, before anything is written) the full build below runs instead.
    int n_static = 1;
    for (int i = 0; i < p.k; ++i) n_static += p.static_widths[i];
    if (n_nodes[seq] == n_static) {
      const int root = emit_tok[(size_t)seq * (ESP_MAX_MASKS + 1) + ne - 1];
      int my_depth = 0, my_j = 0, base = 1;
      for (int i = 1; i <= p.k; ++i) {
        if (tid >= base && tid < base + p.static_widths[i - 1]) { my_depth = i; my_j = tid - base; }
        base += p.static_widths[i - 1];
      }
      const bool live = tid < n_static;
      int ok = 1, par_tok = root, my_tok = root;
      for (int i = 1; i <= p.k && live && my_depth >= i; ++i) {
        const int32_t* li = topk_id + ((size_t)seq * p.k + (i - 1)) * kp;
        const int want = my_depth == i ? my_j : 0;       // own entry at the own depth, the first child above
        int cnt = 0, pick = -1;
        for (int c = 0; c < kp; ++c) {
          const int t = li[c];
          if (t < 0) break;
          if (p.prune_parent && t == par_tok) continue;
          if (p.prune_last && i >= 2 && t == root) continue;
          if (cnt == want) { pick = t; break; }
          ++cnt;
        }
        if (pick < 0) ok = 0;
        if (my_depth == i) my_tok = pick; else par_tok = pick;
      }
      if (!__syncthreads_or(!ok)) {
        if (live) tok[r0 + tid] = my_tok;
        return;
      }
    }
  }
  const int root_tok = emit_tok[(size_t)seq * (ESP_MAX_MASKS + 1) + ne - 1];
  bool odd = false;                     // an entry outside [0, 1], by its bits: above 1, negative or NaN
  for (int t = tid; t < p.k * kp; t += 256) {
    s.list_id[t] = topk_id[(size_t)seq * p.k * kp + t];
    const float q = topk_p[(size_t)seq * p.k * kp + t];
    s.list_p[t] = q;
    odd |= __float_as_uint(q) > __float_as_uint(1.f);
  }
  const bool wave_odd = __builtin_amdgcn_ballot_w64(odd) != 0ull;
  if ((tid & 63) == 0) s.odd[tid >> 6] = wave_odd ? 1 : 0;
  __syncthreads();
  bool wide = false;
  if (__builtin_expect((s.odd[0] | s.odd[1] | s.odd[2] | s.odd[3]) != 0, 0)) {
    bool above = false;                 // among the entries that count
    for (int t = tid; t < p.k * kp; t += 256) {
      const float q = s.list_p[t];
      s.list_p[t] = q > 0.f ? q : (q == q ? 0.f : fabsf(q));   // negative entries count as 0
      above |= t < depth_limit * kp && s.list_id[t] >= 0 && !(q <= 1.f);
    }
    wide = __syncthreads_or(above && !is_static) != 0;
  }
  if (__builtin_expect(wide, 0)) grow_tree<true>(s, p, root_tok, kp, depth_limit);
  else grow_tree<false>(s, p, root_tok, kp, depth_limit);
  __syncthreads();
  if (s.n_keep < 0) {
    if (tid == 0) { n_rows[seq] = 0; n_nodes[seq] = 0; atomicOr(status, ESP_DEV_BAD_TREE); }
    return;
  }
  // rows: the root, then the kept nodes ordered by (depth, creation); one thread per node (at most 255)
  const int n_keep = s.n_keep;
  const int cre = tid < n_keep ? s.cre[s.kept_buf][tid] : 0;
  const uint32_t mine = tid < n_keep ? ((uint32_t)s.dep[cre] << 16) | (uint32_t)cre : 0xffffffffu;
  s.order[tid] = mine;
  if (tid == 0) { s.row_of[0] = 0; s.row_tok[0] = root_tok; s.row_par[0] = -1; s.row_dep[0] = 0; s.orphan = 0; }
  __syncthreads();
  int row = 1;
  for (int b = 0; b < n_keep; b += 4) {
    const u32x4_t o = *reinterpret_cast<const u32x4_t*>(s.order + b);    // entries past n_keep are the largest value
#pragma unroll
    for (int e = 0; e < 4; ++e) row += o[e] < mine ? 1 : 0;
  }
  if (tid < n_keep) {
    s.row_of[cre] = (int16_t)row;
    s.row_tok[row] = s.tok[cre];
    s.row_dep[row] = (int32_t)(mine >> 16);
  }
  __syncthreads();
  // An entry above 1 lets a child outrank its parent, and the cut at B - 1 can then fall between the two: the
  // nodes left are no tree.  All threads agree on that before anything is written; below, every parent row
  // precedes its child's.
  if (tid < n_keep) {
    const int up = s.row_of[s.par[cre]];
    s.row_par[row] = up;
    if (up < 0 || up >= row) s.orphan = 1;
  }
  __syncthreads();
  if (s.orphan) {
    if (tid == 0) { n_rows[seq] = 0; n_nodes[seq] = 0; atomicOr(status, ESP_DEV_BAD_TREE); }
    return;
  }
  if (tid <= n_keep) {
    uint64_t bits[ESP_MAX_TREE_NODES / 64] = {};
    for (int c = tid, hop = 0; c >= 0 && hop <= p.k; c = s.row_par[c], ++hop)   // a node at depth <= k
#pragma unroll
      for (int w = 0; w < ESP_MAX_TREE_NODES / 64; ++w) bits[w] |= (c >> 6) == w ? 1ull << (c & 63) : 0ull;
#pragma unroll
    for (int w = 0; w < ESP_MAX_TREE_NODES / 64; ++w) s.row_anc[tid][w] = bits[w];
    tok[r0 + tid] = s.row_tok[tid];
  }
  if (tid == 0) n_nodes[seq] = n_keep + 1;
  __syncthreads();
  write_rows(seq, rows_per_seq, p.k, p.layout, anc_words, n_keep + 1, ESP_MAX_TREE_NODES / 64,
             [&](int i) { return s.row_par[i]; }, [&](int i) { return s.row_dep[i]; },
             [&](int i, int w) { return s.row_anc[i][w]; }, n_rows, tok, parent, depth, mask_j, attach, anc, status);
}

}  // namespace

// the tree kernels use more dynamic LDS than a kernel gets by default: raise the limits once (also
// called when a context is created, so that no launch inside a stream capture is the first one)
hipError_t tree_prepare() {
  static const hipError_t attr = [] {
    const int from_tree = ESP_MAX_ROWS_PER_SEQ * (8 * (ESP_MAX_ROWS_PER_SEQ / 64) + FROM_TREE_LDS_PER_NODE);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_block_from_tree),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, from_tree);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(k_build_tree), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)sizeof(TreeLds));
  }();
  return attr;
}

hipError_t launch_block_from_tree(hipStream_t st, int batch, int rows_per_seq, int k, int layout, int anc_words,
                                  int32_t* n_rows, const int32_t* n_nodes, int32_t* tok, int32_t* parent,
                                  int32_t* depth, int32_t* mask_j, int32_t* attach, uint64_t* anc,
                                  int32_t* status) {
  const size_t lds = (size_t)rows_per_seq * (8 * anc_words + FROM_TREE_LDS_PER_NODE);
  hipLaunchKernelGGL(k_block_from_tree, dim3(batch), dim3(256), lds, st, rows_per_seq, k, layout, anc_words, n_rows,
                     n_nodes, tok, parent, depth, mask_j, attach, anc, status);
  return hipGetLastError();
}

hipError_t launch_verify_accept(hipStream_t st, int dtype, const BlockDev& b, const KvDev& kv,
                                const int32_t* node_argmax, int n_layers, int n_kv, int hd, int32_t* n_emit,
                                int32_t* emit_tok, int32_t* accepted_row, int32_t* star_row, int32_t* status) {
  (void)status;
  hipLaunchKernelGGL(k_verify, dim3(b.batch), dim3(256), 0, st, b, kv, node_argmax, n_emit, emit_tok,
                     accepted_row, star_row);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  dim3 grid(n_layers * n_kv, b.batch);
  if (dtype == ESP_F32)
    hipLaunchKernelGGL(k_kv_commit<float>, grid, dim3(hd), 0, st, b, kv, n_kv, hd, n_emit, accepted_row);
  else
    hipLaunchKernelGGL(k_kv_commit<bf16_t>, grid, dim3(hd), 0, st, b, kv, n_kv, hd, n_emit, accepted_row);
  return hipGetLastError();
}

hipError_t launch_mask_rows(hipStream_t st, const BlockDev& b, const int32_t* star_row, const int32_t* n_emit,
                            int32_t* a_rows, int32_t* n_lists) {
  hipLaunchKernelGGL(k_mask_rows, dim3(b.batch), dim3(64), 0, st, b, star_row, n_emit, a_rows, n_lists);
  return hipGetLastError();
}

hipError_t launch_build_tree(hipStream_t st, const esp_tree_params& p, int batch, const int32_t* topk_id,
                             const float* topk_p, int kp, const int32_t* n_lists, const int32_t* n_emit,
                             const int32_t* emit_tok, int rows_per_seq, int anc_words, int32_t* n_rows,
                             int32_t* n_nodes, int32_t* tok, int32_t* parent, int32_t* depth, int32_t* mask_j,
                             int32_t* attach, uint64_t* anc, int32_t* status, bool reuse) {
  const hipError_t attr = tree_prepare();
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(k_build_tree, dim3(batch), dim3(256), sizeof(TreeLds), st, p, topk_id, topk_p, kp, n_lists,
                     n_emit, emit_tok, rows_per_seq, anc_words, n_rows, n_nodes, tok, parent, depth, mask_j,
                     attach, anc, status, reuse ? 1 : 0);
  return hipGetLastError();
}
