// Graph encoding and lower-set family construction on the device.
//
// Sets of nodes are bitmasks of `words` 64-bit words (node v is bit v % 64
// of word v / 64).  Per-set work runs one wavefront per set with lane w
// holding word w (at most 64 words, i.e. 4096 nodes), so unions,
// differences and subset tests are single VALU ops per lane and set sums
// are lane-local popcount-style loops followed by a wave reduction.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rc_internal.h"

namespace rcdp {

namespace {

constexpr int kWave = 64;

__device__ __forceinline__ int64_t wave_sum_i64(int64_t x) {
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, kWave);
  return x;
}

__device__ __forceinline__ uint64_t bcast_u64(uint64_t x, int lane) {
  return __shfl(x, lane, kWave);
}

// Sum of c[v] over the set bits of one word (nodes 64*word + bit).
__device__ __forceinline__ int64_t word_cost(uint64_t bits, int word, const int32_t* c) {
  int64_t s = 0;
  while (bits) {
    const int b = __builtin_ctzll(bits);
    s += c[word * 64 + b];
    bits &= bits - 1;
  }
  return s;
}

// ---------------------------------------------------------------- graph

__global__ void k_zero_u64(uint64_t* p, int64_t count) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

// Edge (v, w): bit w in succ[v], bit v in pred[w] (Section 2's delta sets
// of single nodes).  Duplicate edges OR the same bit.
__global__ void k_graph_masks(int n, int words, const int32_t* row_ptr, const int32_t* col_idx,
                              uint64_t* succ, uint64_t* pred) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  for (int e = row_ptr[v]; e < row_ptr[v + 1]; e++) {
    const int w = col_idx[e];
    atomicOr((unsigned long long*)&succ[(int64_t)v * words + (w >> 6)], 1ull << (w & 63));
    atomicOr((unsigned long long*)&pred[(int64_t)w * words + (v >> 6)], 1ull << (v & 63));
  }
}

// ------------------------------------------------------------- ancestors

// L^v = {w : v reachable from w} (Section 4.3) = {v} + union of L^p over the
// predecessors p of v.  Nodes are visited depth by depth (longest path from
// a source), so every predecessor is final before it is read.  One
// workgroup; the closure lives in LDS when it fits.
template <bool kLds>
__global__ __launch_bounds__(1024) void k_ancestors(int n, int words, int num_depths,
                                                    int num_edges, const int32_t* by_depth,
                                                    const int32_t* depth_ptr,
                                                    const int32_t* pred_ptr,
                                                    const int32_t* pred_idx, uint64_t* anc_out) {
  // LDS variant: the ancestor masks, the depth order and the predecessor
  // lists all live in LDS, so each depth costs LDS traffic and one barrier
  extern __shared__ uint64_t lds_anc[];
  uint64_t* anc = kLds ? lds_anc : anc_out;
  int32_t* l_pp = reinterpret_cast<int32_t*>(lds_anc + (kLds ? (int64_t)n * words : 0));
  int32_t* l_pi = l_pp + (n + 1);
  int32_t* l_bd = l_pi + num_edges;
  int32_t* l_dp = l_bd + n;
  if (kLds) {
    for (int x = threadIdx.x; x <= n; x += blockDim.x) l_pp[x] = pred_ptr[x];
    for (int x = threadIdx.x; x < num_edges; x += blockDim.x) l_pi[x] = pred_idx[x];
    for (int x = threadIdx.x; x < n; x += blockDim.x) l_bd[x] = by_depth[x];
    for (int x = threadIdx.x; x <= num_depths; x += blockDim.x) l_dp[x] = depth_ptr[x];
    __syncthreads();
  }
  const int32_t* PP = kLds ? l_pp : pred_ptr;
  const int32_t* PI = kLds ? l_pi : pred_idx;
  const int32_t* BD = kLds ? l_bd : by_depth;
  const int32_t* DP = kLds ? l_dp : depth_ptr;
  for (int d = 0; d < num_depths; d++) {
    const int b = DP[d], e = DP[d + 1];
    const int items = (e - b) * words;
    for (int it = threadIdx.x; it < items; it += blockDim.x) {
      const int v = BD[b + it / words];
      const int w = it % words;
      uint64_t x = (v >> 6) == w ? (1ull << (v & 63)) : 0ull;
      for (int q = PP[v]; q < PP[v + 1]; q++) x |= anc[(int64_t)PI[q] * words + w];
      anc[(int64_t)v * words + w] = x;
    }
    __syncthreads();
  }
  if (kLds) {
    for (int it = threadIdx.x; it < n * words; it += blockDim.x) anc_out[it] = anc[it];
  }
}

// Small graphs: one wave walks the nodes in depth order (a topological
// order) with the masks, the depth order and the predecessor lists in LDS;
// lane w owns word w of every mask.  A node's predecessors are all earlier
// in the order, and one wave's LDS accesses complete in order, so the walk
// needs no barrier at all (the depth-parallel sweep pays one per depth).
__global__ __launch_bounds__(64) void k_ancestors_wave(int n, int words, int num_edges,
                                                       const int32_t* by_depth,
                                                       const int32_t* pred_ptr,
                                                       const int32_t* pred_idx,
                                                       uint64_t* anc_out) {
  extern __shared__ uint64_t lds_anc[];
  uint64_t* anc = lds_anc;
  int32_t* l_pp = reinterpret_cast<int32_t*>(lds_anc + (int64_t)n * words);
  int32_t* l_pi = l_pp + (n + 1);
  int32_t* l_bd = l_pi + num_edges;
  const int lane = threadIdx.x;
  for (int x = lane; x <= n; x += kWave) l_pp[x] = pred_ptr[x];
  for (int x = lane; x < num_edges; x += kWave) l_pi[x] = pred_idx[x];
  for (int x = lane; x < n; x += kWave) l_bd[x] = by_depth[x];
  __syncthreads();
  const bool active = lane < words;
  if (n == 0) return;
  int v = l_bd[0];
  int q0 = l_pp[v], q1 = l_pp[v + 1];
  for (int idx = 0; idx < n; idx++) {
    const int vn = idx + 1 < n ? l_bd[idx + 1] : v;     // the next node, ahead
    uint64_t x = (v >> 6) == lane ? (1ull << (v & 63)) : 0ull;
    int q = q0;
    for (; q + 4 <= q1; q += 4) {
      const int a0 = l_pi[q], a1 = l_pi[q + 1], a2 = l_pi[q + 2], a3 = l_pi[q + 3];
      if (active)
        x |= anc[(int64_t)a0 * words + lane] | anc[(int64_t)a1 * words + lane] |
             anc[(int64_t)a2 * words + lane] | anc[(int64_t)a3 * words + lane];
    }
    for (; q < q1; q++)
      if (active) x |= anc[(int64_t)l_pi[q] * words + lane];
    if (active) anc[(int64_t)v * words + lane] = x;
    q0 = l_pp[vn];
    q1 = l_pp[vn + 1];
    v = vn;
  }
  __syncthreads();
  for (int it = lane; it < n * words; it += kWave) anc_out[it] = anc[it];
}

// Transitive closure of the predecessor relation in one workgroup (graphs
// whose masks fit LDS and have at most kClosureWords words): A[v] starts as
// the direct predecessors of v; for every node k, each mask that contains k
// absorbs A[k] (Warshall's algorithm, any order of k).  The 64 nodes of a
// mask word are taken as one block, so that a block costs four barriers
// instead of a barrier per node:
//  - the block's own rows absorb one another in registers, lane i row
//    64 kb + i, wave w word w beside its own copy of word kb, which says who
//    absorbs whom; row k reaches the other lanes by readlane;
//  - a row outside absorbs the closed rows of the block that it contains, the
//    highest first, and skips those that are below one already taken: with
//    ids in a topological order the block's antichain, not its 64 nodes.
// Then L^v = A[v] + {v}.  Bound by the chain of 64 register steps per word:
// DenseNet-121's 426 nodes 28 us, against 132 with a barrier per node.
constexpr int kClosureWords = 8;
constexpr int kClosureThreads = 1024;
constexpr int kClosureItems = 4;        // items per thread: n * words <= 4096
static_assert(kClosureWords <= kClosureThreads / kWave, "a wave per word");

__device__ __forceinline__ uint64_t readlane_u64(uint64_t x, int l) {
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)x, l);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(x >> 32), l);
  return ((uint64_t)hi << 32) | lo;
}

__global__ __launch_bounds__(kClosureThreads) void k_ancestors_closure(int n, int words,
                                                                       const uint64_t* pred_mask,
                                                                       uint64_t* anc_out) {
  extern __shared__ uint64_t A[];
  const int items = n * words;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  for (int x = threadIdx.x; x < items; x += kClosureThreads) A[x] = pred_mask[x];
  int vw[kClosureItems], wo[kClosureItems];          // row offset v * words and word w
#pragma unroll
  for (int r = 0; r < kClosureItems; r++) {
    const int it = threadIdx.x + r * kClosureThreads;
    const int v = it / words;
    vw[r] = it < items ? v * words : -1;
    wo[r] = it - v * words;
  }
  __syncthreads();
  for (int kb = 0; kb < words; kb++) {
    const int row0 = 64 * kb * words;                   // the block's rows
    const int row1 = min(64 * (kb + 1), n) * words;
    const int own = row0 + lane * words;
    const bool mine = wave < words && own < row1;
    uint64_t x = 0;
    if (wave < words) {
      uint64_t d = mine ? A[own + kb] : 0;
      x = mine ? A[own + wave] : 0;
#pragma unroll
      for (int k = 0; k < 64; k++) {
        if (k % 16 == 0 && row0 + k * words >= row1) break;   // lanes past the last row hold 0
        const uint64_t take = 0 - (d >> k & 1);
        x |= readlane_u64(x, k) & take;
        d |= readlane_u64(d, k) & take;
      }
    }
    __syncthreads();
    if (mine) A[own + wave] = x;
    __syncthreads();
    uint64_t acc[kClosureItems];
#pragma unroll
    for (int r = 0; r < kClosureItems; r++) {
      acc[r] = 0;
      if (vw[r] < 0 || (vw[r] >= row0 && vw[r] < row1)) continue;
      uint64_t left = A[vw[r] + kb];
      while (left) {
        const int j = 63 - __builtin_clzll(left);
        const uint64_t* const aj = A + row0 + j * words;
        acc[r] |= aj[wo[r]];
        left &= ~(aj[kb] | 1ull << j);
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kClosureItems; r++)
      if (acc[r]) A[vw[r] + wo[r]] |= acc[r];
    __syncthreads();
  }
  for (int x = threadIdx.x; x < items; x += kClosureThreads) {
    const int v = x / words, w = x - v * words;
    anc_out[x] = A[x] | ((v >> 6) == w ? 1ull << (v & 63) : 0ull);
  }
}

// ---------------------------------------------------- exact enumeration

// Reverse search over lower sets, one size level after the other.  A lower
// set X != {} has the canonical parent X \ {x}, x the largest node id of X
// with no successor inside X (removing such an x keeps delta^-(X \ {x})
// inside).  For every parent P of size s and node v with v not in P and
// delta^-(v) inside P, the child X = P + {v} is kept iff v is X's canonical
// element.  With S(P) the nodes of P without a successor in P, those of X
// are S(X) = (S(P) \ delta^-(v)) + {v} (no node of P has v's successors: a
// successor of v inside P would put v in P), so v is canonical iff no node
// of S(P) \ delta^-(v) has a larger id.  S travels with each candidate
// (top), and a test costs a few words instead of a walk over P's nodes.
// Children are appended through an atomic counter; their order within the
// level is fixed afterwards by the rank kernel.  Level s is
// cand[lvl[s] .. lvl[s] + cnt[s]).
//
// Word w of the test of (P, v): bit 1 = a predecessor of v is missing, bit 2
// = a node of S(P) \ delta^-(v) above v, bit 4 = v is in P.
__device__ __forceinline__ int enum_word(uint64_t Pw, uint64_t Sw, uint64_t pred, int w, int v) {
  const int vw = v >> 6;
  const uint64_t vb = w == vw ? 1ull << (v & 63) : 0ull;
  const uint64_t above = w > vw ? ~0ull : (w == vw ? ~((vb << 1) - 1) : 0ull);
  return ((pred & ~Pw) != 0 ? 1 : 0) | ((Sw & ~pred & above) != 0 ? 2 : 0) |
         ((Pw & vb) != 0 ? 4 : 0);
}

// The first levels in one workgroup, while the frontier fits LDS (frontier
// sets x words <= kEnumWords) and its level is at most kEnumWork word tests
// (sets x nodes x words, sixteen a thread): two barriers a level instead of
// two launches.  Small graphs end here: a 16-node chain, 16 levels, 14 us
// against 60, the 40-node ladder's 40 levels 37 us against 247.  A larger
// level is faster over the whole chip.  Whole builds with the limit at 8 K /
// 16 K / 32 K / 64 K / 128 K tests / LDS alone, in us: two chains of 60 nodes
// (levels of up to 15 K tests) 575 / 559 / 555 / 556 / 559 / 571; of 100 (81
// K) 1605 / 1613 / 1659 / 2053 / 3071 / 3100; of 150 (226 K) 4532 / 4562 /
// 4537 / 4687 / 5581 / 11664; the antichain of 12 (11 K) 207 / 184 / 183 /
// 183 / 182 / 187.  stop[0] = the first level not expanded (n when done),
// stop[1] = sets found, stop[2] = overflow (host memory).
constexpr int kEnumWords = 1024;
constexpr int64_t kEnumWork = 16384;
constexpr int kEnumMasks = 3072;          // n * words of the graphs taken
constexpr int kEnumThreads = 1024;

__global__ __launch_bounds__(kEnumThreads) void k_enum_block(int n, int words,
                                                             const uint64_t* pred_g,
                                                             uint64_t* cand, uint64_t* top,
                                                             int64_t cap, int32_t* lvl,
                                                             int32_t* cnt, DevStatus* st,
                                                             int32_t* stop) {
  __shared__ uint64_t s_pred[kEnumMasks];
  __shared__ uint64_t s_set[2][kEnumWords], s_top[2][kEnumWords];
  __shared__ int32_t s_n[2];
  const int tid = threadIdx.x;
  for (int x = tid; x < (int)(sizeof(DevStatus) / 4); x += kEnumThreads)
    reinterpret_cast<int32_t*>(st)[x] = 0;
  for (int x = tid; x < n * words; x += kEnumThreads) s_pred[x] = pred_g[x];
  for (int x = tid; x < n + 2; x += kEnumThreads) cnt[x] = 0;
  for (int x = tid; x < words; x += kEnumThreads) {
    s_set[0][x] = 0;
    s_top[0][x] = 0;
    cand[x] = 0;                          // the empty set
    top[x] = 0;
  }
  if (tid == 0) s_n[0] = 1;
  __syncthreads();
  int64_t base = 0;                       // first set of the level
  int lev = 0, here = 1;
  bool over = false;
  for (; lev < n; lev++) {
    const int f = lev & 1;
    if (tid == 0) {
      s_n[f ^ 1] = 0;
      lvl[lev] = (int32_t)base;
      cnt[lev] = here;
    }
    __syncthreads();
    const uint32_t items = (uint32_t)here * (uint32_t)n;
    for (uint32_t it = tid; it < items; it += kEnumThreads) {
      const int p = (int)(it / (uint32_t)n), v = (int)(it - (uint32_t)p * n);
      int bad = 0;
      for (int w = 0; w < words; w++)
        bad |= enum_word(s_set[f][p * words + w], s_top[f][p * words + w], s_pred[v * words + w],
                         w, v);
      if (bad) continue;
      const int slot = atomicAdd(&s_n[f ^ 1], 1);
      const int64_t g = base + here + slot;
      for (int w = 0; w < words; w++) {
        const uint64_t vb = w == (v >> 6) ? 1ull << (v & 63) : 0ull;
        const uint64_t X = s_set[f][p * words + w] | vb;
        const uint64_t S = (s_top[f][p * words + w] & ~s_pred[v * words + w]) | vb;
        if ((slot + 1) * words <= kEnumWords) {
          s_set[f ^ 1][slot * words + w] = X;
          s_top[f ^ 1][slot * words + w] = S;
        }
        if (g < cap) {
          cand[g * words + w] = X;
          top[g * words + w] = S;
        }
      }
    }
    __syncthreads();
    const int next = s_n[f ^ 1];
    base += here;
    here = next;
    over = base + here > cap;
    if (over || here * words > kEnumWords || (int64_t)here * n * words > kEnumWork) {
      lev++;
      break;
    }
  }
  if (tid == 0) {
    lvl[lev] = (int32_t)base;
    cnt[lev] = over ? 0 : here;
    lvl[lev + 1] = (int32_t)(base + here);
    st->count = over ? cap : base + here;
    st->overflow = over;
    stop[0] = over ? n : lev;
    stop[1] = over ? 0 : (int32_t)(base + here);
    stop[2] = over;
  }
}

// One size level over the whole chip; cnt[s + 1] starts at 0.
__global__ __launch_bounds__(256) void k_enum_level(int n, int words, int s, const uint64_t* pred,
                                                    uint64_t* cand, uint64_t* top, int64_t cap,
                                                    int32_t* lvl, int32_t* cnt, DevStatus* st) {
  const int64_t pb = lvl[s];
  const int32_t here = (int32_t)max((int64_t)0, min((int64_t)cnt[s], cap - pb));  // stored sets
  const int64_t nb = pb + here;            // first set of the next level
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    lvl[s + 1] = (int32_t)nb;
    st->count = nb;                        // the last level's own launch adds nothing
  }
  const uint32_t items = (uint32_t)here * (uint32_t)n;     // at most 65535 * 4096
  for (uint32_t it = blockIdx.x * blockDim.x + threadIdx.x; it < items;
       it += gridDim.x * blockDim.x) {
    const uint32_t p = it / (uint32_t)n;
    const int v = (int)(it - p * (uint32_t)n);
    const uint64_t* P = cand + (pb + p) * words;
    const uint64_t* S = top + (pb + p) * words;
    const uint64_t* pv = pred + (int64_t)v * words;
    int bad = 0;
    for (int w = 0; w < words && !bad; w++) bad = enum_word(P[w], S[w], pv[w], w, v);
    if (bad) continue;
    const int64_t g = nb + atomicAdd(&cnt[s + 1], 1);
    if (g >= cap) {
      st->overflow = 1;
      continue;
    }
    for (int w = 0; w < words; w++) {
      const uint64_t vb = w == (v >> 6) ? 1ull << (v & 63) : 0ull;
      cand[g * words + w] = P[w] | vb;
      top[g * words + w] = (S[w] & ~pv[w]) | vb;
    }
  }
}

// The empty set as level 0, for graphs that k_enum_block does not take.
__global__ void k_enum_start(int n, int words, uint64_t* cand, uint64_t* top, int32_t* lvl,
                             int32_t* cnt, DevStatus* st) {
  for (int x = threadIdx.x; x < (int)(sizeof(DevStatus) / 4); x += blockDim.x)
    reinterpret_cast<int32_t*>(st)[x] = 0;
  for (int w = threadIdx.x; w < words; w += blockDim.x) {
    cand[w] = 0;
    top[w] = 0;
  }
  for (int x = threadIdx.x; x < n + 2; x += blockDim.x) cnt[x] = x == 0 ? 1 : 0;
  if (threadIdx.x == 0) lvl[0] = 0;
}

// The size of the enumerated family to the host.
__global__ void k_enum_end(int n, const int32_t* lvl, const int32_t* cnt, DevStatus* st,
                           int32_t* stop) {
  const int32_t total = lvl[n] + cnt[n];
  st->count = total;
  stop[0] = n;
  stop[1] = total;
  stop[2] = st->overflow;
}

// --------------------------------------------------------------- ranking

// Numeric comparison of two sets stored set-major (most significant word
// first): -1, 0, 1.
__device__ __forceinline__ int cmp_value(const uint64_t* a, const uint64_t* b, int words) {
  for (int w = words - 1; w >= 0; w--)
    if (a[w] != b[w]) return a[w] < b[w] ? -1 : 1;
  return 0;
}

// Canonical order: ascending size, then ascending numeric value.  Exact
// family: candidates are grouped by size level (reverse search yields no
// duplicates) and ranked within their level, a wave per candidate with the
// level's other sets over its lanes (6199 sets in levels of up to 583: 10 us
// against 132 with a thread per candidate).  Output is word-major:
// bits[w * fstride + index].
__global__ __launch_bounds__(256) void k_rank(int words, int64_t F, const uint64_t* cand,
                                              const int32_t* lvl, const int32_t* cnt,
                                              uint64_t* bits, int64_t fstride, DevStatus* st) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t x = blockIdx.x * (int64_t)(blockDim.x / kWave) + threadIdx.x / kWave;
  if (x >= F) return;
  const uint64_t* X = cand + x * words;
  int sz = lane < words ? __popcll(X[lane]) : 0;
  for (int off = 32; off > 0; off >>= 1) sz += __shfl_xor(sz, off, kWave);
  const int64_t b = lvl[sz], e = b + cnt[sz];
  int less = 0;
  for (int64_t y = b + lane; y < e; y += kWave)
    less += cmp_value(cand + y * words, X, words) < 0 ? 1 : 0;
  for (int off = 32; off > 0; off >>= 1) less += __shfl_xor(less, off, kWave);
  const int64_t rank = b + less;
  if (rank >= fstride) {
    if (lane == 0) st->error = 1;
    return;
  }
  if (lane < words) bits[(int64_t)lane * fstride + rank] = X[lane];
}

// Pruned family: candidates are [0] the empty set, [1..n] the sets L^v
// (pairwise distinct), [n+1] V, which is dropped when some L^v already
// equals V.  One workgroup: the candidates are bucketed by size (a counting
// sort in LDS), and a candidate's index is the number of candidates of
// smaller size plus those of its own size with a smaller numeric value.
// anc[v] = L^v; the empty set and V are formed here.  Clears the status.
__global__ __launch_bounds__(1024) void k_rank_pruned(int words, int n, const uint64_t* anc,
                                                      uint64_t* bits, int64_t fstride,
                                                      DevStatus* st) {
  constexpr int kThreads = 1024;
  __shared__ int32_t s_sz[kMaxNodes + 2];
  __shared__ int32_t s_start[kMaxNodes + 2];   // candidates of size < s, s = 0..n+1
  __shared__ int32_t s_next[kMaxNodes + 2];    // next free slot of each size's bucket
  __shared__ int32_t s_list[kMaxNodes + 2];    // candidates grouped by size
  __shared__ int32_t s_wsum[kThreads / kWave];
  __shared__ int32_t s_vdup;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  const int total = n + 2, bins = n + 2;       // sizes 0..n, counted one bin up
  auto word = [&](int x, int w) -> uint64_t {
    if (x == 0) return 0;
    if (x <= n) return anc[(int64_t)(x - 1) * words + w];
    const int left = n - w * 64;
    return left >= 64 ? ~0ull : (1ull << left) - 1;
  };
  if (tid < (int)(sizeof(DevStatus) / 4)) reinterpret_cast<int32_t*>(st)[tid] = 0;
  if (tid == 0) s_vdup = n == 0;                 // V is the empty set itself
  for (int x = tid; x < bins; x += kThreads) s_start[x] = 0;
  for (int x = tid; x < total; x += kThreads) {
    int c = 0;
    for (int w = 0; w < words; w++) c += __popcll(word(x, w));
    s_sz[x] = c;
  }
  __syncthreads();
  for (int x = 1 + tid; x <= n; x += kThreads)
    if (s_sz[x] == n) s_vdup = 1;                 // some L^v is V already
  __syncthreads();
  const int valid = s_vdup ? n + 1 : n + 2;
  for (int x = tid; x < valid; x += kThreads) atomicAdd(&s_start[s_sz[x] + 1], 1);
  __syncthreads();
  // inclusive scan of the counts: s_start[s] = candidates of size < s
  const int per = (bins + kThreads - 1) / kThreads;
  const int b0 = min(bins, tid * per), b1 = min(bins, b0 + per);
  int run = 0;
  for (int q = b0; q < b1; q++) {
    run += s_start[q];
    s_start[q] = run;
  }
  int incl = run;
  for (int off = 1; off < kWave; off <<= 1) {
    const int y = __shfl_up(incl, off, kWave);
    if (lane >= off) incl += y;
  }
  if (lane == kWave - 1) s_wsum[wave] = incl;
  __syncthreads();
  int before = incl - run;
  for (int q = 0; q < wave; q++) before += s_wsum[q];
  for (int q = b0; q < b1; q++) {
    s_start[q] += before;
    s_next[q] = s_start[q];
  }
  __syncthreads();
  for (int x = tid; x < valid; x += kThreads) s_list[atomicAdd(&s_next[s_sz[x]], 1)] = x;
  __syncthreads();
  for (int x = tid; x < valid; x += kThreads) {
    const int sx = s_sz[x];
    int64_t rank = s_start[sx];
    for (int q = s_start[sx]; q < s_start[sx + 1]; q++) {
      const int y = s_list[q];
      if (y == x) continue;
      int w = words - 1;
      while (w > 0 && word(y, w) == word(x, w)) w--;
      if (word(y, w) < word(x, w)) rank++;
    }
    if (rank >= fstride) {
      st->error = 1;
      continue;
    }
    for (int w = 0; w < words; w++) bits[(int64_t)w * fstride + rank] = word(x, w);
  }
  if (tid == 0) st->count = valid;
}

// ------------------------------------------------------- per-set values

// Per set L (one wave, lane w = word w):
//   boundary(L) = {v in L : some successor of v outside L}  (Section 2)
//   T(L), M(L), T(boundary), M(boundary)
//   A(L) = M(delta+(L) \ L) + M(delta-(delta+(L) \ L) \ L), the terms (iii)
//   and (iv) of Eq. 2 for the set L' = L (for a lower set L the
//   predecessors of delta+(L) inside L add nothing outside L)
//   w_L = T(L \ boundary(L)) + 1, the cells of row L that can be finite.
template <bool kLds>
__global__ __launch_bounds__(256) void k_set_quantities(
    int64_t F, int n, int words, int64_t fstride, const uint64_t* bits, const uint64_t* succ_g,
    const uint64_t* pred_g, const int32_t* T, const int32_t* M, uint64_t* bd, int32_t* size,
    int32_t* Tsum, int32_t* Msum, int32_t* Tbd, int32_t* Mbd, int32_t* A, int32_t* w_out) {
  // small graphs: the successor and predecessor masks of every node in LDS
  extern __shared__ uint64_t lds_nb[];
  const uint64_t* succ = succ_g;
  const uint64_t* pred = pred_g;
  if (kLds) {
    const int64_t cnt = (int64_t)n * words;
    for (int64_t x = threadIdx.x; x < cnt; x += blockDim.x) {
      lds_nb[x] = succ_g[x];
      lds_nb[cnt + x] = pred_g[x];
    }
    __syncthreads();
    succ = lds_nb;
    pred = lds_nb + cnt;
  }
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t s = blockIdx.x * (int64_t)(blockDim.x / kWave) + threadIdx.x / kWave;
  if (s >= F) return;
  const bool active = lane < words;
  const uint64_t L = active ? bits[(int64_t)lane * fstride + s] : 0ull;
  uint64_t out = 0, bdw = 0;
  for (int ww = 0; ww < words; ww++) {
    uint64_t Lw = bcast_u64(L, ww);
    while (Lw) {
      const int v = ww * 64 + __builtin_ctzll(Lw);
      Lw &= Lw - 1;
      const uint64_t sv = active ? succ[(int64_t)v * words + lane] : 0ull;
      out |= sv;
      const bool leaves = __any((sv & ~L) != 0);
      if (leaves && lane == ww) bdw |= 1ull << (v & 63);
    }
  }
  out &= ~L;
  uint64_t in2 = 0;
  for (int ww = 0; ww < words; ww++) {
    uint64_t Ow = bcast_u64(out, ww);
    while (Ow) {
      const int v = ww * 64 + __builtin_ctzll(Ow);
      Ow &= Ow - 1;
      if (active) in2 |= pred[(int64_t)v * words + lane];
    }
  }
  in2 &= ~L;
  const int64_t tl = wave_sum_i64(active ? word_cost(L, lane, T) : 0);
  const int64_t ml = wave_sum_i64(active ? word_cost(L, lane, M) : 0);
  const int64_t tb = wave_sum_i64(active ? word_cost(bdw, lane, T) : 0);
  const int64_t mb = wave_sum_i64(active ? word_cost(bdw, lane, M) : 0);
  const int64_t ao = wave_sum_i64(active ? word_cost(out, lane, M) : 0);
  const int64_t ai = wave_sum_i64(active ? word_cost(in2, lane, M) : 0);
  const int sz = (int)wave_sum_i64(active ? __popcll(L) : 0);
  if (active) bd[(int64_t)lane * fstride + s] = bdw;
  if (lane == 0) {
    size[s] = sz;
    Tsum[s] = (int32_t)tl;
    Msum[s] = (int32_t)ml;
    Tbd[s] = (int32_t)tb;
    Mbd[s] = (int32_t)mb;
    A[s] = (int32_t)(ao + ai);
    w_out[s] = (int32_t)(tl - tb + 1);
  }
}

// The same quantities for graphs of at most kLaneWords * 64 nodes, with the
// nodes spread over the lanes instead of walked one by one: lane l takes
// node 64 ww + l of every word ww, ORs its successor (then predecessor)
// words into kLaneWords register accumulators and adds its costs; word w
// of a union is then one wave OR reduction, a sum one wave sum.
constexpr int kLaneWords = 8;

__device__ __forceinline__ uint64_t wave_or_u64(uint64_t x) {
  for (int off = 32; off > 0; off >>= 1) x |= __shfl_xor(x, off, kWave);
  return x;
}

template <bool kLds>
__global__ __launch_bounds__(256) void k_set_quantities_lanes(
    int64_t F, int n, int words, int64_t fstride, const uint64_t* bits, const uint64_t* succ_g,
    const uint64_t* pred_g, const int32_t* T, const int32_t* M, uint64_t* bd, int32_t* size,
    int32_t* Tsum, int32_t* Msum, int32_t* Tbd, int32_t* Mbd, int32_t* A, int32_t* w_out) {
  extern __shared__ uint64_t lds_nb[];
  const uint64_t* succ = succ_g;
  const uint64_t* pred = pred_g;
  if (kLds) {
    const int64_t cnt = (int64_t)n * words;
    for (int64_t x = threadIdx.x; x < cnt; x += blockDim.x) {
      lds_nb[x] = succ_g[x];
      lds_nb[cnt + x] = pred_g[x];
    }
    __syncthreads();
    succ = lds_nb;
    pred = lds_nb + cnt;
  }
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t s = blockIdx.x * (int64_t)(blockDim.x / kWave) + threadIdx.x / kWave;
  if (s >= F) return;
  // word w of L on lane w, and every word of L in scalars
  const uint64_t L = lane < words ? bits[(int64_t)lane * fstride + s] : 0ull;
  uint64_t Lw[kLaneWords];
#pragma unroll
  for (int w = 0; w < kLaneWords; w++) Lw[w] = w < words ? readlane_u64(L, w) : 0ull;

  // delta+(L) \ L and the boundary: lane l walks nodes 64 ww + l of L
  uint64_t acc[kLaneWords];
#pragma unroll
  for (int w = 0; w < kLaneWords; w++) acc[w] = 0;
  uint64_t bdw = 0;                                   // boundary word `lane`
  int64_t tl = 0, ml = 0, tb = 0, mb = 0;
#pragma unroll
  for (int ww = 0; ww < kLaneWords; ww++) {
    if (ww >= words) break;
    const int v = ww * 64 + lane;
    const bool in = (Lw[ww] >> lane) & 1ull;
    bool leaves = false;
#pragma unroll
    for (int w = 0; w < kLaneWords; w++) {
      if (w >= words) break;
      const uint64_t x = in ? succ[(int64_t)v * words + w] & ~Lw[w] : 0ull;
      acc[w] |= x;
      leaves |= x != 0;
    }
    const uint64_t bmask = __ballot(in && leaves);
    if (lane == ww) bdw = bmask;
    if (in) {
      const int32_t tv = T[v], mv = M[v];
      tl += tv;
      ml += mv;
      if (leaves) {
        tb += tv;
        mb += mv;
      }
    }
  }
  uint64_t out = 0;                                   // word `lane` of delta+(L) \ L
#pragma unroll
  for (int w = 0; w < kLaneWords; w++) {
    if (w >= words) break;
    const uint64_t r = wave_or_u64(acc[w]);
    if (lane == w) out = r;
  }
  // delta-(delta+(L) \ L) \ L, and M of both sets
#pragma unroll
  for (int w = 0; w < kLaneWords; w++) acc[w] = 0;
  int64_t ao = 0;
#pragma unroll
  for (int ww = 0; ww < kLaneWords; ww++) {
    if (ww >= words) break;
    const int v = ww * 64 + lane;
    const bool in = (readlane_u64(out, ww) >> lane) & 1ull;
    if (!in) continue;
    ao += M[v];
#pragma unroll
    for (int w = 0; w < kLaneWords; w++) {
      if (w >= words) break;
      acc[w] |= pred[(int64_t)v * words + w] & ~Lw[w];
    }
  }
  int64_t ai = 0;
#pragma unroll
  for (int w = 0; w < kLaneWords; w++) {
    if (w >= words) break;
    const uint64_t in2w = wave_or_u64(acc[w]);        // word w, the same on every lane
    if ((in2w >> lane) & 1ull) ai += M[w * 64 + lane];
  }
  tl = wave_sum_i64(tl);
  ml = wave_sum_i64(ml);
  tb = wave_sum_i64(tb);
  mb = wave_sum_i64(mb);
  ao = wave_sum_i64(ao);
  ai = wave_sum_i64(ai);
  const int sz = (int)wave_sum_i64(lane < words ? __popcll(L) : 0);
  if (lane < words) bd[(int64_t)lane * fstride + s] = bdw;
  if (lane == 0) {
    size[s] = sz;
    Tsum[s] = (int32_t)tl;
    Msum[s] = (int32_t)ml;
    Tbd[s] = (int32_t)tb;
    Mbd[s] = (int32_t)mb;
    A[s] = (int32_t)(ao + ai);
    w_out[s] = (int32_t)(tl - tb + 1);
  }
}

// ------------------------------------------------------------------ pairs

// Subset test of family members i and j (word-major storage).
__device__ __forceinline__ bool is_subset(const uint64_t* bits, int64_t fstride, int words,
                                          int64_t i, int64_t j) {
  for (int w = 0; w < words; w++)
    if (bits[(int64_t)w * fstride + i] & ~bits[(int64_t)w * fstride + j]) return false;
  return true;
}

// Predecessors of target j: i < j with L_i a proper subset of L_j.  The
// family is sorted by size, so every proper subset has a smaller index;
// equal sizes are never proper subsets.  counts[j] = their number, walg[j] =
// the sum of their w_i (relaxations of Algorithm 1's loop), and with mask
// [F][mw] (mw = ceil(F / 64); null: not kept) their bits, which k_pair_write
// reads instead of testing the subsets again.
__global__ __launch_bounds__(256) void k_pair_count(int64_t F, int words, int64_t fstride,
                                                    const uint64_t* __restrict__ bits,
                                                    const int32_t* __restrict__ size,
                                                    const int32_t* __restrict__ w, int64_t* counts,
                                                    int64_t* walg, uint64_t* mask, int64_t mw) {
  const int64_t j = blockIdx.x;
  __shared__ int64_t s_c[4], s_w[4];
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  int64_t c = 0, ws = 0;
  const int sj = size[j];
  for (int64_t i0 = 0; i0 < j; i0 += blockDim.x) {
    const int64_t i = i0 + threadIdx.x;
    const bool is = i < j && size[i] < sj && is_subset(bits, fstride, words, i, j);
    const uint64_t b = __ballot(is);
    if (mask && lane == 0 && i < j) mask[j * mw + i / kWave] = b;
    if (is) {
      c++;
      ws += w[i];
    }
  }
  c = wave_sum_i64(c);
  ws = wave_sum_i64(ws);
  if (lane == 0) {
    s_c[wv] = c;
    s_w[wv] = ws;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    counts[j] = s_c[0] + s_c[1] + s_c[2] + s_c[3];
    walg[j] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
  }
}

// Pair data of (L = L_i, L' = L_j), in ascending i for every target j:
//   dt = T((L' \ L) \ bd(L')) = T(L' \ bd(L')) - T(L) + T(L & bd(L'))
//   dm = M(bd(L') \ L)        = M(bd(L')) - M(L & bd(L'))
//   c  = 2 M(L' \ L) + A(L')  = 2 (M(L') - M(L)) + A(L')
// so that the step of Algorithm 1 from (L, t, m) is admitted iff
// m + c <= B and then lands on (L', t + dt) with cache m + dm.  Only the
// two sums over L & bd(L') depend on the pair; bd(L') is small: its nodes,
// the same for every pair of the workgroup, are walked with their costs in
// scalars while each thread tests its own L_i.  kMask: the pairs come from
// k_pair_count's bits (prefix of their counts in LDS, no barrier per chunk),
// and sp gets, per target, its first pair from the sets of the block of
// `rows` targets before its own, and from its own block (two block sizes; a
// null array is not wanted).
struct PairSplit {
  int32_t rows[2];
  int64_t* split[2];
};
constexpr int64_t kMaskSets = 8192;      // families whose pair bits are kept (8 MB)

template <bool kMask>
__global__ __launch_bounds__(256) void k_pair_write(
    int64_t F, int words, int64_t fstride, const uint64_t* __restrict__ bits,
    const uint64_t* __restrict__ bd, const int32_t* __restrict__ size,
    const int32_t* __restrict__ Tsum, const int32_t* __restrict__ Msum,
    const int32_t* __restrict__ Tbd, const int32_t* __restrict__ Mbd,
    const int32_t* __restrict__ A, const int32_t* __restrict__ T, const int32_t* __restrict__ M,
    const int64_t* __restrict__ pred_ptr, const uint64_t* __restrict__ mask, int64_t mw,
    int32_t* pidx, int32_t* pdt, int32_t* pdm, int32_t* pc, PairSplit sp) {
  const int64_t j = blockIdx.x;
  __shared__ int64_t base;
  __shared__ int32_t wave_cnt[4];
  __shared__ int32_t s_pre[kMask ? kMaskSets / kWave + 1 : 1];
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  const int64_t p0 = pred_ptr[j];
  if (kMask) {
    // exclusive prefix of the mask words' counts, wave 0
    if (wv == 0) {
      const int nw = (int)((j + kWave - 1) / kWave);
      int run = 0;
      for (int x0 = 0; x0 < nw; x0 += kWave) {
        const int x = x0 + lane;
        const int v = x < nw ? __popcll(mask[j * mw + x]) : 0;
        int incl = v;
        for (int off = 1; off < kWave; off <<= 1) {
          const int y = __shfl_up(incl, off, kWave);
          if (lane >= off) incl += y;
        }
        if (x < nw) s_pre[x] = run + incl - v;
        run += __shfl(incl, kWave - 1, kWave);
      }
    }
  } else if (threadIdx.x == 0) {
    base = p0;
  }
  __syncthreads();
  if (kMask && threadIdx.x < 4 && j > 0 && sp.split[threadIdx.x / 2]) {
    // first pair from the previous block's sets, and from the block's own
    const int32_t rows = sp.rows[threadIdx.x / 2];
    const int64_t j0 = 1 + (j - 1) / rows * rows;
    const int64_t x = threadIdx.x % 2 == 0 ? max((int64_t)0, j0 - rows) : j0;
    const uint64_t below = x / kWave * kWave < j
                               ? mask[j * mw + x / kWave] & ((1ull << (x & (kWave - 1))) - 1)
                               : 0ull;
    const int nw = (int)((j + kWave - 1) / kWave);
    sp.split[threadIdx.x / 2][2 * j + threadIdx.x % 2] =
        x / kWave < nw ? p0 + s_pre[x / kWave] + __popcll(below) : pred_ptr[j + 1];
  }
  const int sj = size[j];
  const int64_t tj = (int64_t)Tsum[j] - Tbd[j], mbj = Mbd[j], cj = 2 * (int64_t)Msum[j] + A[j];
  for (int64_t i0 = 0; i0 < j; i0 += blockDim.x) {
    const int64_t i = i0 + threadIdx.x;
    bool is;
    int64_t p = 0;
    if (kMask) {
      const uint64_t b = i < j ? mask[j * mw + i / kWave] : 0ull;
      is = (b >> lane) & 1;
      if (is) p = p0 + s_pre[i / kWave] + __popcll(b & ((1ull << lane) - 1));
    } else {
      is = i < j && size[i] < sj && is_subset(bits, fstride, words, i, j);
      const uint64_t b = __ballot(is);
      if (lane == 0) wave_cnt[wv] = __popcll(b);
      __syncthreads();
      p = base + __popcll(b & ((1ull << lane) - 1));
      for (int q = 0; q < wv; q++) p += wave_cnt[q];
    }
    if (__any(is)) {
      int64_t ti = 0, mi = 0;
      for (int ww = 0; ww < words; ww++) {
        uint64_t Bw = bd[(int64_t)ww * fstride + j];
        if (!Bw) continue;
        const uint64_t x = is ? bits[(int64_t)ww * fstride + i] : 0ull;
        for (; Bw; Bw &= Bw - 1) {
          const int v = __builtin_ctzll(Bw);
          const int64_t hit = -(int64_t)((x >> v) & 1);
          ti += hit & T[ww * 64 + v];
          mi += hit & M[ww * 64 + v];
        }
      }
      if (is) {
        pidx[p] = (int32_t)i;
        pdt[p] = (int32_t)(tj - Tsum[i] + ti);
        pdm[p] = (int32_t)(mbj - mi);
        pc[p] = (int32_t)(cj - 2 * (int64_t)Msum[i]);
      }
    }
    if (!kMask) {
      __syncthreads();
      if (threadIdx.x == 0)
        for (int q = 0; q < (int)(blockDim.x / kWave); q++) base += wave_cnt[q];
      __syncthreads();
    }
  }
}

// ------------------------------------------------------------ scan / sum

// Sum over the workgroup's lanes before this one, and the workgroup's total.
constexpr int kScanThreads = 1024;
__device__ __forceinline__ int64_t block_scan(int64_t x, int64_t* s_part, int64_t* total) {
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  int64_t incl = x;
  for (int off = 1; off < kWave; off <<= 1) {
    const int64_t y = __shfl_up(incl, off, kWave);
    if (lane >= off) incl += y;
  }
  if (lane == kWave - 1) s_part[wv] = incl;
  __syncthreads();
  int64_t before = 0, all = 0;
  for (int q = 0; q < kScanThreads / kWave; q++) {
    const int64_t v = s_part[q];
    if (q < wv) before += v;
    all += v;
  }
  __syncthreads();
  *total = all;
  return before + incl - x;
}

// Exclusive scan of in[0..count) into out[0..count]; one workgroup.
__global__ __launch_bounds__(kScanThreads) void k_scan(const int64_t* in, int64_t* out,
                                                       int64_t count) {
  __shared__ int64_t s_part[kScanThreads / kWave];
  int64_t carry = 0;
  for (int64_t b = 0; b < count; b += kScanThreads) {
    const int64_t i = b + threadIdx.x;
    int64_t total;
    const int64_t pre = block_scan(i < count ? in[i] : 0, s_part, &total);
    if (i < count) out[i] = carry + pre;
    carry += total;
  }
  if (threadIdx.x == 0) out[count] = carry;
}

// The family's shape in one launch: row offsets (rows right-aligned inside
// their padded slots: row s ends on a kRowAlign boundary, so every column
// counted from the row end is made of whole 128-byte lines, and at least
// kGuard padding cells separate it from the previous row), predecessor
// offsets, the relaxation count, and what the host needs of them, written
// straight to its pinned buffer (the status, sizes, widths, both offset
// arrays and M(L) at the byte offsets of o).
struct ShapeOut {
  char* host;
  int64_t o_st, o_size, o_w, o_off, o_pp, o_msum;
};

__global__ __launch_bounds__(kScanThreads) void k_shape(int64_t F, const int32_t* size,
                                                        const int32_t* w, const int32_t* Msum,
                                                        const int64_t* counts,
                                                        const int64_t* walg, int64_t* row_off,
                                                        int64_t* pred_ptr, DevStatus* st,
                                                        ShapeOut o) {
  __shared__ int64_t s_part[kScanThreads / kWave];
  int32_t* h_size = reinterpret_cast<int32_t*>(o.host + o.o_size);
  int32_t* h_w = reinterpret_cast<int32_t*>(o.host + o.o_w);
  int32_t* h_msum = reinterpret_cast<int32_t*>(o.host + o.o_msum);
  int64_t* h_off = reinterpret_cast<int64_t*>(o.host + o.o_off);
  int64_t* h_pp = reinterpret_cast<int64_t*>(o.host + o.o_pp);
  int64_t cells = 0, pairs = 0, relax = 0;
  for (int64_t b = 0; b < F; b += kScanThreads) {
    const int64_t i = b + threadIdx.x;
    const int32_t wi = i < F ? w[i] : 0;
    const int64_t slot = i < F ? row_slot(wi) : 0;
    int64_t total;
    const int64_t off = cells + block_scan(slot, s_part, &total) + slot - wi;
    cells += total;
    const int64_t pp = pairs + block_scan(i < F ? counts[i] : 0, s_part, &total);
    pairs += total;
    block_scan(i < F ? walg[i] : 0, s_part, &total);
    relax += total;
    if (i < F) {
      row_off[i] = off;
      pred_ptr[i] = pp;
      h_off[i] = off;
      h_pp[i] = pp;
      h_size[i] = size[i];
      h_w[i] = wi;
      h_msum[i] = Msum[i];
    }
  }
  if (threadIdx.x == 0) {
    row_off[F] = cells;
    pred_ptr[F] = pairs;
    h_off[F] = cells;
    h_pp[F] = pairs;
    st->walg = relax;
    DevStatus x = *st;
    x.walg = relax;
    *reinterpret_cast<DevStatus*>(o.host + o.o_st) = x;
  }
}

}  // namespace

// ============================================================== launchers

hipError_t launch_graph_masks(rc_graph g, const int32_t* d_row_ptr, const int32_t* d_col_idx,
                              hipStream_t s) {
  const int64_t cnt = 2 * (int64_t)g->n * g->words;      // dPred follows dSucc
  hipLaunchKernelGGL(k_zero_u64, dim3(64), dim3(256), 0, s, g->dSucc, cnt);
  hipLaunchKernelGGL(k_graph_masks, dim3((g->n + 255) / 256), dim3(256), 0, s, g->n, g->words,
                     d_row_ptr, d_col_idx, g->dSucc, g->dPred);
  return hipGetLastError();
}

hipError_t launch_ancestors(rc_graph g, uint64_t* anc, hipStream_t s) {
  const size_t lds_closure = sizeof(uint64_t) * (size_t)g->n * g->words;
  if (g->words <= kClosureWords && (int64_t)g->n * g->words <= kClosureItems * kClosureThreads) {
    hipLaunchKernelGGL(k_ancestors_closure, dim3(1), dim3(kClosureThreads), lds_closure, s, g->n,
                       g->words, g->dPred, anc);
    return hipGetLastError();
  }
  const size_t lds_wave = sizeof(uint64_t) * (size_t)g->n * g->words +
                          sizeof(int32_t) * ((size_t)g->n + 1 + g->num_pred_edges + g->n);
  if (lds_wave <= 64 * 1024) {
    hipLaunchKernelGGL(k_ancestors_wave, dim3(1), dim3(kWave), lds_wave, s, g->n, g->words,
                       g->num_pred_edges, g->dByDepth, g->dPredPtr, g->dPredIdx, anc);
    return hipGetLastError();
  }
  const size_t lds = sizeof(uint64_t) * (size_t)g->n * g->words +
                     sizeof(int32_t) * ((size_t)g->n + 1 + g->num_pred_edges + g->n +
                                        g->num_depths + 1);
  if (lds <= 64 * 1024) {
    hipLaunchKernelGGL(k_ancestors<true>, dim3(1), dim3(1024), lds, s, g->n, g->words,
                       g->num_depths, g->num_pred_edges, g->dByDepth, g->dDepthPtr, g->dPredPtr,
                       g->dPredIdx, anc);
  } else {
    hipLaunchKernelGGL(k_ancestors<false>, dim3(1), dim3(1024), 0, s, g->n, g->words,
                       g->num_depths, g->num_pred_edges, g->dByDepth, g->dDepthPtr, g->dPredPtr,
                       g->dPredIdx, anc);
  }
  return hipGetLastError();
}

// Sets of the exact family, grouped by size; stop (host memory, 3 words): the
// first level not expanded, the number of sets, overflow.  first: level to
// start from (0, or stop[0] of the call before).
hipError_t launch_enum_exact(rc_graph g, int32_t first, uint64_t* cand, uint64_t* top, int64_t cap,
                             int32_t* lvl, int32_t* cnt, DevStatus* st, int32_t* stop,
                             hipStream_t s) {
  if (first == 0 && g->words <= kMaxWords / 8 && (int64_t)g->n * g->words <= kEnumMasks) {
    hipLaunchKernelGGL(k_enum_block, dim3(1), dim3(kEnumThreads), 0, s, g->n, g->words, g->dPred,
                       cand, top, cap, lvl, cnt, st, stop);
    return hipGetLastError();
  }
  if (first == 0)
    hipLaunchKernelGGL(k_enum_start, dim3(1), dim3(64), 0, s, g->n, g->words, cand, top, lvl, cnt,
                       st);
  for (int lev = first; lev < g->n; lev++)
    hipLaunchKernelGGL(k_enum_level, dim3(512), dim3(256), 0, s, g->n, g->words, lev, g->dPred,
                       cand, top, cap, lvl, cnt, st);
  hipLaunchKernelGGL(k_enum_end, dim3(1), dim3(1), 0, s, g->n, lvl, cnt, st, stop);
  return hipGetLastError();
}

hipError_t launch_rank_exact(rc_family f, const uint64_t* cand, const int32_t* lvl,
                             const int32_t* cnt, hipStream_t s) {
  const int per_block = 256 / kWave;
  hipLaunchKernelGGL(k_rank, dim3((unsigned)((f->F + per_block - 1) / per_block)), dim3(256), 0, s,
                     f->g->words, f->F, cand, lvl, cnt, f->bits, f->fstride, f->status);
  return hipGetLastError();
}

hipError_t launch_rank_pruned(rc_family f, hipStream_t s) {
  rc_graph g = f->g;
  hipLaunchKernelGGL(k_rank_pruned, dim3(1), dim3(1024), 0, s, g->words, g->n, g->dAnc, f->bits,
                     f->fstride, f->status);
  return hipGetLastError();
}

hipError_t launch_set_quantities(rc_family f, hipStream_t s) {
  rc_graph g = f->g;
  const int per_block = 256 / kWave;
  const dim3 grid((unsigned)((f->F + per_block - 1) / per_block));
  const size_t lds = 2 * sizeof(uint64_t) * (size_t)g->n * g->words;
  if (g->words <= kLaneWords) {
    if (lds <= 64 * 1024)
      hipLaunchKernelGGL(k_set_quantities_lanes<true>, grid, dim3(256), lds, s, f->F, g->n,
                         g->words, f->fstride, f->bits, g->dSucc, g->dPred, g->dT, g->dM, f->bd,
                         f->size, f->Tsum, f->Msum, f->Tbd, f->Mbd, f->A, f->w);
    else
      hipLaunchKernelGGL(k_set_quantities_lanes<false>, grid, dim3(256), 0, s, f->F, g->n,
                         g->words, f->fstride, f->bits, g->dSucc, g->dPred, g->dT, g->dM, f->bd,
                         f->size, f->Tsum, f->Msum, f->Tbd, f->Mbd, f->A, f->w);
    return hipGetLastError();
  }
  if (lds <= 64 * 1024)
    hipLaunchKernelGGL(k_set_quantities<true>, grid, dim3(256), lds, s, f->F, g->n, g->words,
                       f->fstride, f->bits, g->dSucc, g->dPred, g->dT, g->dM, f->bd, f->size,
                       f->Tsum, f->Msum, f->Tbd, f->Mbd, f->A, f->w);
  else
    hipLaunchKernelGGL(k_set_quantities<false>, grid, dim3(256), 0, s, f->F, g->n, g->words,
                       f->fstride, f->bits, g->dSucc, g->dPred, g->dT, g->dM, f->bd, f->size,
                       f->Tsum, f->Msum, f->Tbd, f->Mbd, f->A, f->w);
  return hipGetLastError();
}

// 64-bit words of the pair bits of one target; 0: they are not kept.
int64_t pair_mask_words(rc_family f) { return f->F <= kMaskSets ? (f->F + kWave - 1) / kWave : 0; }

hipError_t launch_pair_count(rc_family f, int64_t* counts, int64_t* walg, uint64_t* mask,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_pair_count, dim3((unsigned)f->F), dim3(256), 0, s, f->F, f->g->words,
                     f->fstride, f->bits, f->size, f->w, counts, walg, mask, pair_mask_words(f));
  return hipGetLastError();
}

hipError_t launch_shape(rc_family f, const int64_t* counts, const int64_t* walg, char* host,
                        const int64_t (&o)[6], hipStream_t s) {
  hipLaunchKernelGGL(k_shape, dim3(1), dim3(kScanThreads), 0, s, f->F, f->size, f->w, f->Msum,
                     counts, walg, f->row_off, f->pred_ptr, f->status,
                     ShapeOut{host, o[0], o[1], o[2], o[3], o[4], o[5]});
  return hipGetLastError();
}

hipError_t launch_scan(const int64_t* in, int64_t* out, int64_t count, hipStream_t s) {
  hipLaunchKernelGGL(k_scan, dim3(1), dim3(kScanThreads), 0, s, in, out, count);
  return hipGetLastError();
}

hipError_t launch_pair_write(rc_family f, const uint64_t* mask, hipStream_t s) {
  rc_graph g = f->g;
  const int64_t mw = pair_mask_words(f);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)f->F), dim3(256), 0, s, f->F, g->words, f->fstride,
                       f->bits, f->bd, f->size, f->Tsum, f->Msum, f->Tbd, f->Mbd, f->A, g->dT,
                       g->dM, f->pred_ptr, mask, mw, f->pidx, f->pdt, f->pdm, f->pc,
                       PairSplit{{f->dual_rows, block_fill_rows()}, {f->dual_split, f->fb_split}});
  };
  if (mask)
    go(k_pair_write<true>);
  else
    go(k_pair_write<false>);
  return hipGetLastError();
}

}  // namespace rcdp
