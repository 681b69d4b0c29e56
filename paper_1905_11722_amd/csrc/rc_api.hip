// Host side of the C ABI declared in include/rc.h: argument validation,
// device memory plumbing and kernel orchestration.  Every step of the
// method itself runs in the kernels of graph.hip, family.hip and fill.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <utility>
#include <vector>

#include "rc_internal.h"
#include "dual.h"
#include "schedule.h"

using namespace rcdp;

#define RC_HIP(x)                                     \
  do {                                                \
    hipError_t e_ = (x);                              \
    if (e_ != hipSuccess) {                           \
      rcdp::set_last_error(#x, e_);                   \
      return RC_E_DEVICE;                             \
    }                                                 \
  } while (0)

namespace rcdp {

static thread_local char g_last_error[512] = "";

void set_last_error(const char* what, hipError_t e) {
  std::snprintf(g_last_error, sizeof(g_last_error), "%s: %s", what, hipGetErrorString(e));
}

void set_last_error_msg(const char* msg) {
  std::snprintf(g_last_error, sizeof(g_last_error), "%s", msg);
}

int32_t jitter_seed() {
  const char* env = std::getenv("RCDP_JITTER");
  return env ? (int32_t)std::strtol(env, nullptr, 10) : 0;
}

namespace {
// Free pinned buffers, smallest first: a request takes the smallest that
// fits, or allocates a power of two of at least 64 KB.  Never destroyed, so
// that no buffer is released after the runtime has shut down.
struct StagingPool {
  std::mutex mu;
  std::vector<std::pair<size_t, char*>> free_list;
};
StagingPool& staging_pool() {
  static StagingPool* pool = new StagingPool();
  return *pool;
}
}  // namespace

Staging::Staging(size_t bytes) {
  StagingPool& pool = staging_pool();
  {
    std::lock_guard<std::mutex> lock(pool.mu);
    auto& fl = pool.free_list;
    for (size_t x = 0; x < fl.size(); x++) {
      if (fl[x].first >= bytes) {
        n_ = fl[x].first;
        p_ = fl[x].second;
        fl.erase(fl.begin() + (std::ptrdiff_t)x);
        return;
      }
    }
  }
  size_t n = (size_t)64 << 10;
  while (n < bytes) n <<= 1;
  void* p = nullptr;
  if (hipHostMalloc(&p, n, hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) {
    (void)hipGetLastError();               // no launch after it has failed
    return;
  }
  p_ = static_cast<char*>(p);
  n_ = n;
}

Staging::~Staging() {
  if (!p_ || pending_) return;
  StagingPool& pool = staging_pool();
  std::lock_guard<std::mutex> lock(pool.mu);
  auto& fl = pool.free_list;
  auto it = fl.begin();
  while (it != fl.end() && it->first < n_) ++it;
  fl.insert(it, {n_, p_});
}

// Sizes of the memory-indexed table of one solve (rc_solve_dual): argument
// checks, the effective budget, the row width and the scratch it needs.
int dual_buffers(rc_family f, int64_t B, int32_t objective, DualBuffers* out) {
  if (!f || B < 0) return RC_E_ARG;
  if (objective != RC_TIME_CENTRIC && objective != RC_MEMORY_CENTRIC) return RC_E_ARG;
  const int64_t Beff = std::min<int64_t>(B, 2 * f->g->M_total);
  const int64_t W = std::min<int64_t>(Beff, f->g->M_total) + 1;
  if (f->g->T_total >= (int64_t)UINT32_MAX || W > INT32_MAX / 2 ||
      (double)f->F * (double)W > (double)((int64_t)1 << 31))
    return RC_E_OVERFLOW;
  *out = DualBuffers();
  out->Beff = Beff;
  out->W = W;
  out->cells = f->F * W;
  return RC_OK;
}

// The memory-indexed table, its selection and (when any schedule output is
// asked for) its traceback, in the device buffers of b; results to the host
// outputs.  Synchronises s.  e0 / e1 (may be null) bracket the table's
// kernels.  Allocates nothing.
int dual_solve(rc_family f, int32_t objective, const DualBuffers& b, hipEvent_t e0,
               hipEvent_t e1, hipStream_t s, int64_t* t_opt, int64_t* m_opt, int32_t* k,
               int32_t* chain_host, int32_t* seg_host, uint8_t* cached_host, int64_t* overhead,
               int64_t* peak, int64_t* cache_mem) {
  const bool pinned = b.host != nullptr;
  if (pinned) b.host->in_flight();
  const hipError_t le = launch_dual(f, f->level_pairs, (int32_t)b.Beff, (int32_t)b.W, objective,
                                    b.D, b.st, pinned ? &b.host_st[0] : nullptr, e0, e1, s);
  if (le != hipSuccess) {
    set_last_error("dual table launch", le);
    return RC_E_DEVICE;
  }
  DevStatus hs;
  if (!pinned) RC_HIP(hipMemcpyAsync(&hs, b.st, sizeof(hs), hipMemcpyDeviceToHost, s));
  RC_HIP(hipStreamSynchronize(s));
  if (pinned) hs = b.host_st[0];
  const bool schedule = k || chain_host || seg_host || cached_host || overhead || peak || cache_mem;
  if (schedule && hs.t_sel >= 0) {
    const size_t n = (size_t)f->g->n;
    const ScheduleOut out{b.out_chain, b.seg, b.cached, pinned ? &b.host_st[1] : b.st};
    const hipError_t te = launch_dual_trace(f, (int32_t)b.Beff, (int32_t)b.W, objective, b.D,
                                            b.st, b.chain, out, s);
    if (te != hipSuccess) {
      set_last_error("dual traceback launch", te);
      return RC_E_DEVICE;
    }
    DevStatus ts;
    if (!pinned) RC_HIP(hipMemcpyAsync(&ts, b.st, sizeof(ts), hipMemcpyDeviceToHost, s));
    RC_HIP(hipStreamSynchronize(s));
    if (pinned) ts = b.host_st[1];
    if (ts.error || ts.k < 0 || ts.k > f->F) {
      set_last_error_msg("dual traceback: the walk did not end at (empty set, 0, 0)");
      return RC_E_DEVICE;
    }
    auto bring = [&](void* dst, const void* src, size_t bytes) -> int {
      if (!dst || bytes == 0) return RC_OK;
      if (pinned)
        std::memcpy(dst, src, bytes);
      else
        RC_HIP(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s));
      return RC_OK;
    };
    if (bring(chain_host, b.out_chain, sizeof(int32_t) * (size_t)ts.k) != RC_OK ||
        bring(seg_host, b.seg, sizeof(int32_t) * n) != RC_OK ||
        bring(cached_host, b.cached, n) != RC_OK)
      return RC_E_DEVICE;
    if (!pinned) RC_HIP(hipStreamSynchronize(s));
    if (k) *k = ts.k;
    if (overhead) *overhead = ts.overhead;
    if (peak) *peak = ts.peak;
    if (cache_mem) *cache_mem = ts.cache_mem;
  }
  if (pinned) b.host->landed();
  if (t_opt) *t_opt = hs.t_sel;
  if (m_opt) *m_opt = hs.t_sel >= 0 ? hs.m_sel : -1;
  return hs.t_sel >= 0 ? RC_OK : RC_INFEASIBLE;
}

void* Arena::raw(size_t bytes) {
  void* p = nullptr;
  if (alloc) {
    p = alloc(bytes, user);
  } else if (hipMalloc(&p, bytes) != hipSuccess) {
    (void)hipGetLastError();               // no launch after it has failed
    p = nullptr;
  }
  if (p) ptrs.push_back(p);
  return p;
}

// Small buffers are carved from chunks of kChunk bytes, so that a handle
// costs a few calls of the caller's allocator rather than one per buffer.
void* Arena::get(size_t bytes) {
  if (bytes == 0) bytes = 1;
  bytes = (bytes + 255) & ~size_t(255);
  if (bytes > kChunk / 4) return raw(bytes);
  if (cur + bytes > end) {
    char* c = static_cast<char*>(raw(kChunk));
    if (!c) return nullptr;
    cur = c;
    end = c + kChunk;
  }
  void* p = cur;
  cur += bytes;
  return p;
}

void Arena::release_all() {
  cur = end = nullptr;
  for (void* p : ptrs) {
    if (alloc) {
      if (free_fn) free_fn(p, user);
    } else {
      (void)hipFree(p);
    }
  }
  ptrs.clear();
}

}  // namespace rcdp

static hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

extern "C" {

const char* rc_last_error(void) { return g_last_error; }

const char* rc_status_str(int status) {
  switch (status) {
    case RC_OK: return "ok";
    case RC_INFEASIBLE: return "infeasible: no chain of lower sets meets the budget";
    case RC_E_ARG: return "invalid argument";
    case RC_E_CYCLE: return "the graph has a directed cycle or a self-loop";
    case RC_E_COST: return "a node cost is not positive";
    case RC_E_TOO_MANY_SETS: return "the lower-set family exceeds max_sets";
    case RC_E_OVERFLOW: return "a value exceeds the table's integer widths";
    case RC_E_NOMEM: return "device allocation failed";
    case RC_E_DEVICE: return "HIP runtime or kernel error";
    case RC_E_STATE: return "handle in the wrong state";
    case RC_E_SCRATCH: return "the solve needs more than the allocation-free scratch";
    default: return "unknown status";
  }
}

// ------------------------------------------------------------------ graph

int rc_graph_create(int32_t n, const int32_t* row_ptr, const int32_t* col_idx, const int32_t* T,
                    const int32_t* M, rc_alloc_fn alloc, rc_free_fn free_fn, void* user,
                    void* stream, rc_graph* out) {
  if (!out || n < 0 || n > kMaxNodes) return RC_E_ARG;
  if (n > 0 && (!row_ptr || !T || !M)) return RC_E_ARG;
  if (alloc && !free_fn) return RC_E_ARG;
  // -- validation of the CSR and costs (Section 2: T_v > 0, M_v > 0)
  int64_t nnz = 0;
  if (n > 0) {
    if (row_ptr[0] != 0) return RC_E_ARG;
    for (int v = 0; v < n; v++)
      if (row_ptr[v + 1] < row_ptr[v]) return RC_E_ARG;
    nnz = row_ptr[n];
    if (nnz > 0 && !col_idx) return RC_E_ARG;
    for (int64_t e = 0; e < nnz; e++)
      if (col_idx[e] < 0 || col_idx[e] >= n) return RC_E_ARG;
  }
  int64_t Ttot = 0, Mtot = 0;
  for (int v = 0; v < n; v++) {
    if (T[v] < 1 || M[v] < 1) return RC_E_COST;
    Ttot += T[v];
    Mtot += M[v];
  }
  if (Ttot >= (int64_t)INT32_MAX - 1 || Mtot >= ((int64_t)1 << 29)) return RC_E_OVERFLOW;
  // -- deduplicated predecessor lists and topological depth (Kahn by levels)
  std::vector<std::vector<int32_t>> preds(n);
  for (int v = 0; v < n; v++) {
    for (int64_t e = row_ptr[v]; e < row_ptr[v + 1]; e++) {
      int w = col_idx[e];
      if (w == v) return RC_E_CYCLE;
      preds[w].push_back(v);
    }
  }
  for (auto& p : preds) {
    std::sort(p.begin(), p.end());
    p.erase(std::unique(p.begin(), p.end()), p.end());
  }
  std::vector<int32_t> indeg(n), depth(n, 0), order;
  order.reserve(n);
  std::vector<std::vector<int32_t>> succs(n);
  for (int w = 0; w < n; w++)
    for (int v : preds[w]) succs[v].push_back(w);
  for (int v = 0; v < n; v++) {
    indeg[v] = (int32_t)preds[v].size();
    if (indeg[v] == 0) order.push_back(v);
  }
  for (size_t q = 0; q < order.size(); q++) {
    int v = order[q];
    for (int w : succs[v]) {
      depth[w] = std::max(depth[w], depth[v] + 1);
      if (--indeg[w] == 0) order.push_back(w);
    }
  }
  if ((int)order.size() != n) return RC_E_CYCLE;
  int32_t D = 0;
  for (int v = 0; v < n; v++) D = std::max(D, depth[v] + 1);
  std::vector<int32_t> by_depth(n), depth_ptr(D + 1, 0);
  for (int v = 0; v < n; v++) depth_ptr[depth[v] + 1]++;
  for (int d = 0; d < D; d++) depth_ptr[d + 1] += depth_ptr[d];
  {
    std::vector<int32_t> fill(depth_ptr.begin(), depth_ptr.end() - 1);
    for (int v = 0; v < n; v++) by_depth[fill[depth[v]]++] = v;
  }
  std::vector<int32_t> pred_ptr(n + 1, 0), pred_idx;
  for (int v = 0; v < n; v++) {
    pred_ptr[v + 1] = pred_ptr[v] + (int32_t)preds[v].size();
    pred_idx.insert(pred_idx.end(), preds[v].begin(), preds[v].end());
  }

  rc_graph g = new (std::nothrow) rc_graph_s();
  if (!g) return RC_E_NOMEM;
  g->n = n;
  g->words = (n + 63) / 64;
  g->T_total = Ttot;
  g->M_total = Mtot;
  g->arena.alloc = alloc;
  g->arena.free_fn = free_fn;
  g->arena.user = user;
  g->num_depths = D;
  for (int v = 0; v < n; v++) g->num_sinks += succs[v].empty() ? 1 : 0;
  hipStream_t s = as_stream(stream);
  int st = RC_OK;
  // every array through one pinned buffer and one copy (eight copies from
  // pageable memory waited for one after the other); one copy from pageable
  // memory where no pinned memory can be had
  int32_t *d_row_ptr = nullptr, *d_col_idx = nullptr;
  StageLayout lay;
  const size_t o_T = lay.add<int32_t>(n), o_M = lay.add<int32_t>(n),
               o_pp = lay.add<int32_t>(n + 1),
               o_pi = lay.add<int32_t>((int64_t)pred_idx.size()), o_bd = lay.add<int32_t>(n),
               o_dp = lay.add<int32_t>(D + 1), o_rp = lay.add<int32_t>(n + 1),
               o_ci = lay.add<int32_t>(nnz);
  Staging stage(lay.bytes);
  std::vector<char> pageable(stage.data() ? 0 : lay.bytes);
  char* const host = stage.data() ? stage.data() : pageable.data();
  char* dev = static_cast<char*>(g->arena.get(lay.bytes));
  if (!dev) st = RC_E_NOMEM;
  g->num_pred_edges = (int32_t)pred_idx.size();
  if (st == RC_OK) {
    auto put = [&](size_t off, const int32_t* from, int64_t count) {
      if (count > 0) std::memcpy(host + off, from, sizeof(int32_t) * (size_t)count);
      return reinterpret_cast<int32_t*>(dev + off);
    };
    g->dT = put(o_T, T, n);
    g->dM = put(o_M, M, n);
    g->dPredPtr = put(o_pp, pred_ptr.data(), n + 1);
    g->dPredIdx = put(o_pi, pred_idx.data(), (int64_t)pred_idx.size());
    g->dByDepth = put(o_bd, by_depth.data(), n);
    g->dDepthPtr = put(o_dp, depth_ptr.data(), D + 1);
    d_row_ptr = put(o_rp, row_ptr, row_ptr && n > 0 ? n + 1 : 0);
    d_col_idx = put(o_ci, col_idx, nnz);
    stage.in_flight();
    if (hipMemcpyAsync(dev, host, lay.bytes, hipMemcpyHostToDevice, s) != hipSuccess)
      st = RC_E_DEVICE;
  }
  if (st == RC_OK) {
    g->dSucc = g->arena.get_n<uint64_t>(2 * (int64_t)n * g->words);
    g->dPred = g->dSucc + (int64_t)n * g->words;
    g->dAnc = g->arena.get_n<uint64_t>((int64_t)n * g->words);
    if (!g->dSucc || !g->dAnc) st = RC_E_NOMEM;
  }
  if (st == RC_OK && n > 0 && launch_graph_masks(g, d_row_ptr, d_col_idx, s) != hipSuccess)
    st = RC_E_DEVICE;
  // the ancestor sets (Section 4.3's generators of the pruned family) are a
  // property of the graph: computed once here, read by every pruned family
  if (st == RC_OK && n > 0 && launch_ancestors(g, g->dAnc, s) != hipSuccess) st = RC_E_DEVICE;
  if (st == RC_OK && hipStreamSynchronize(s) != hipSuccess) st = RC_E_DEVICE;
  if (st == RC_OK) stage.landed();
  if (st != RC_OK) {
    (void)hipStreamSynchronize(s);
    g->arena.release_all();
    delete g;
    return st;
  }
  *out = g;
  return RC_OK;
}

void rc_graph_free(rc_graph g) {
  if (!g) return;
  (void)hipDeviceSynchronize();
  g->arena.release_all();
  delete g;
}

// ----------------------------------------------------------------- family

// Which blocks the family's wavefront records use.  RCDP_FILL=wavefront
// forces the row-push fill's fixed blocks and RCDP_FILL=ghost the ghost-zone
// blocks (families of at most kGhostMaxSets sets).  Otherwise: fixed blocks,
// so that the split-panel fill can take the family, for families beyond that
// size, for rows of 2^16 cells and more and for families of kWideMinSets sets
// and more (measured faster than the ghost-zone fill on every such shape
// here, resnet50_t10's 175 sets included: the ghost blocks hold fewer rows,
// so that each staged window serves fewer targets); ghost-zone blocks for
// the smaller families.
static int32_t family_block_kind(rc_family f) {
  const int64_t F = f->F;
  if (F < 2) return 0;
  const char* env = std::getenv("RCDP_FILL");
  if (F > kGhostMaxSets ||
      (env && (std::strcmp(env, "wavefront") == 0 || std::strcmp(env, "wide") == 0)))
    return kBlocksFixed;
  if (env && std::strcmp(env, "ghost") == 0) return kBlocksGhost;
  return f->max_row >= 65536 || F >= kWideMinSets ? kBlocksFixed : kBlocksGhost;
}

// Block starts of the chosen kind (host).
static void cut_blocks(rc_family f, const std::vector<int32_t>& near_h) {
  f->bstart_host.clear();
  if (f->blk_kind == kBlocksGhost) {
    f->bstart_host = ghost_cut(f->F, near_h);
    return;
  }
  for (int64_t j = 1; j < f->F; j += kJB) f->bstart_host.push_back((int32_t)j);
  f->bstart_host.push_back((int32_t)f->F);
}

// Block starts to the device (through pinned memory), then the number of
// panel sources per block and their offsets (rec_ptr).  Uses the family
// arena; counts is scratch of at least nblk + 1 entries.  The staging
// buffer must stay alive until the stream has been synchronised.
static int upload_blocks(rc_family f, int64_t* counts, std::unique_ptr<Staging>& stage,
                         hipStream_t s) {
  Arena& A = f->arena;
  f->nblk = (int64_t)f->bstart_host.size() - 1;
  if (f->nblk <= 0) {
    f->nblk = 0;
    return RC_OK;
  }
  f->bstart = A.get_n<int32_t>(f->nblk + 1);
  f->rec_ptr = A.get_n<int64_t>(f->nblk + 1);
  if (!f->bstart || !f->rec_ptr) return RC_E_NOMEM;
  const size_t bytes = sizeof(int32_t) * (size_t)(f->nblk + 1);
  stage.reset(new (std::nothrow) Staging(bytes));
  if (!stage || !stage->data()) return RC_E_NOMEM;
  std::memcpy(stage->data(), f->bstart_host.data(), bytes);
  stage->in_flight();
  if (hipMemcpyAsync(f->bstart, stage->data(), bytes, hipMemcpyHostToDevice, s) != hipSuccess ||
      launch_blk_count(f, f->nblk, counts, s) != hipSuccess ||
      launch_scan(counts, f->rec_ptr, f->nblk, s) != hipSuccess)
    return RC_E_DEVICE;
  return RC_OK;
}

// Sets of the pruned family: the n ancestor sets L^v (distinct, since v is
// the one maximal node of L^v), the empty set, and V unless V is one of the
// L^v, which happens exactly when the graph has a single sink (every node
// then reaches it).
static int64_t pruned_family_size(rc_graph g) {
  if (g->n == 0) return 1;
  return (int64_t)g->n + 1 + (g->num_sinks > 1 ? 1 : 0);
}

// Record buffers up to this many records are sized from an upper bound
// (every record holds at least one pair) without waiting for their count.
constexpr int64_t kRecordBound = (int64_t)1 << 18;

static int sync_landed(Staging& st, hipStream_t s) {
  if (hipStreamSynchronize(s) != hipSuccess) {
    set_last_error_msg("stream synchronisation failed");
    return RC_E_DEVICE;
  }
  st.landed();
  return RC_OK;
}

static int ensure_records(rc_family f, hipStream_t s);
static int launch_fill_choice(rc_family f);

static int build_family_impl(rc_family f, int64_t max_sets, hipStream_t s) {
  rc_graph g = f->g;
  const int n = g->n, words = g->words;
  Arena& A = f->arena;
  Arena tmp;                       // scratch released at the end of the build
  tmp.alloc = A.alloc;
  tmp.free_fn = A.free_fn;
  tmp.user = A.user;
  struct TmpGuard {
    Arena& a;
    hipStream_t s;
    ~TmpGuard() {
      (void)hipStreamSynchronize(s);
      a.release_all();
    }
  } guard{tmp, s};
  // Kernels write what the host reads into pinned buffers; a build waits for
  // the stream for the family's size (exact family only, once more for a
  // level too large for one workgroup), for its shape, and at the end.

  f->status = A.get_n<DevStatus>(1);
  if (!f->status) return RC_E_NOMEM;

  // ---- a2: the family as bitmasks, in canonical order
  const bool pruned = f->mode == RC_FAMILY_PRUNED;
  int64_t F = 0;
  if (pruned) {
    F = pruned_family_size(g);          // checked against the device's count below
    f->fstride = (int64_t)n + 2;
    f->bits = A.get_n<uint64_t>(f->fstride * words);
    if (!f->bits) return RC_E_NOMEM;
    RC_HIP(launch_rank_pruned(f, s));
  } else {
    const int64_t cap = max_sets;
    uint64_t* cand = tmp.get_n<uint64_t>(cap * words);
    uint64_t* top = tmp.get_n<uint64_t>(cap * words);
    int32_t* lvl = tmp.get_n<int32_t>(n + 3);
    int32_t* cnt = tmp.get_n<int32_t>(n + 3);
    Staging st0(3 * sizeof(int32_t));
    if (!cand || !top || !lvl || !cnt || !st0.data()) return RC_E_NOMEM;
    int32_t* stop = st0.at<int32_t>(0);
    for (int32_t first = 0;;) {
      st0.in_flight();
      RC_HIP(launch_enum_exact(g, first, cand, top, cap, lvl, cnt, f->status, stop, s));
      const int ss = sync_landed(st0, s);
      if (ss != RC_OK) return ss;
      if (stop[2]) return RC_E_TOO_MANY_SETS;
      first = stop[0];
      if (first >= n) break;
    }
    F = stop[1];
    if (F < 1 || F > max_sets) return RC_E_TOO_MANY_SETS;
    f->F = F;
    f->fstride = F;
    f->bits = A.get_n<uint64_t>(F * words);
    if (!f->bits) return RC_E_NOMEM;
    RC_HIP(launch_rank_exact(f, cand, lvl, cnt, s));
  }
  if (F < 1 || F > max_sets) return RC_E_TOO_MANY_SETS;
  f->F = F;

  // ---- a3: per-set quantities
  f->size = A.get_n<int32_t>(F);
  f->Tsum = A.get_n<int32_t>(F);
  f->Msum = A.get_n<int32_t>(F);
  f->Tbd = A.get_n<int32_t>(F);
  f->Mbd = A.get_n<int32_t>(F);
  f->A = A.get_n<int32_t>(F);
  f->w = A.get_n<int32_t>(F);
  f->bd = A.get_n<uint64_t>(f->fstride * words);
  f->row_off = A.get_n<int64_t>(F + 1);
  f->pred_ptr = A.get_n<int64_t>(F + 1);
  int64_t* counts = tmp.get_n<int64_t>(F);
  int64_t* walg = tmp.get_n<int64_t>(F);
  const int64_t mw = pair_mask_words(f);
  uint64_t* mask = mw > 0 ? tmp.get_n<uint64_t>(F * mw) : nullptr;
  if (!f->size || !f->Tsum || !f->Msum || !f->Tbd || !f->Mbd || !f->A || !f->w || !f->bd ||
      !f->row_off || !f->pred_ptr || !counts || !walg || (mw > 0 && !mask))
    return RC_E_NOMEM;
  RC_HIP(launch_set_quantities(f, s));
  // ---- a4: predecessor pairs, counted per target; row and pair offsets
  RC_HIP(launch_pair_count(f, counts, walg, mask, s));
  StageLayout L1;
  const size_t o_st = L1.add<DevStatus>(1), o_size = L1.add<int32_t>(F),
               o_w = L1.add<int32_t>(F), o_off = L1.add<int64_t>(F + 1),
               o_pp = L1.add<int64_t>(F + 1), o_ms = L1.add<int32_t>(F);
  {
    Staging st1(L1.bytes);
    if (!st1.data()) return RC_E_NOMEM;
    const int64_t o[6] = {(int64_t)o_st,  (int64_t)o_size, (int64_t)o_w,
                          (int64_t)o_off, (int64_t)o_pp,   (int64_t)o_ms};
    st1.in_flight();
    RC_HIP(launch_shape(f, counts, walg, st1.data(), o, s));
    const int ss = sync_landed(st1, s);
    if (ss != RC_OK) return ss;
    const DevStatus& h1 = *st1.at<DevStatus>(o_st);
    if (h1.error) return RC_E_DEVICE;
    if (h1.count != F) {
      set_last_error_msg("family build: the device counted another family size");
      return RC_E_DEVICE;
    }
    f->relax = h1.walg;
    const int32_t* size_h = st1.at<int32_t>(o_size);
    const int32_t* w_h = st1.at<int32_t>(o_w);
    const int64_t* off_h = st1.at<int64_t>(o_off);
    const int64_t* pp_h = st1.at<int64_t>(o_pp);
    f->w_host.assign(w_h, w_h + F);
    f->row_off_host.assign(off_h, off_h + F + 1);
    f->cells = off_h[F];
    f->cells_alloc = f->cells + kGuard;
    f->P = pp_h[F];
    if (f->P < 0 || f->P >= ((int64_t)1 << 40) || f->cells >= ((int64_t)1 << 40))
      return RC_E_OVERFLOW;
    f->level_ptr.clear();
    f->level_maxw.clear();
    f->max_row = 0;
    for (int64_t i = 0; i < F; i++) {
      if (i == 0 || size_h[i] != size_h[i - 1]) {
        f->level_ptr.push_back(i);
        f->level_maxw.push_back(0);
      }
      f->level_maxw.back() = std::max(f->level_maxw.back(), w_h[i]);
      f->max_row = std::max<int64_t>(f->max_row, w_h[i]);
    }
    f->level_ptr.push_back(F);
    // the most pairs of a target per size level (the memory-indexed table
    // runs that many pairs per level launch)
    f->level_pairs.clear();
    for (size_t l = 0; l + 1 < f->level_ptr.size(); l++) {
      int64_t most = 0;
      for (int64_t j = f->level_ptr[l]; j < f->level_ptr[l + 1]; j++)
        most = std::max(most, pp_h[j + 1] - pp_h[j]);
      f->level_pairs.push_back(most);
    }
    f->block_pairs = 0;
    for (int64_t j = 1; j < F; j += kJB)
      f->block_pairs = std::max(f->block_pairs, pp_h[std::min<int64_t>(j + kJB, F)] - pp_h[j]);
    if (mask) {
      f->dual_rows = dual_block_rows(F, st1.at<int32_t>(o_ms), &f->dual_halo);
      if (f->cells_alloc < (int64_t)1 << 30) block_fill_halos(f);
    }
  }

  // ---- a4: the pairs themselves
  const int64_t P = f->P;
  if (f->dual_rows > 0) {
    f->dual_split = A.get_n<int64_t>(2 * F);
    if (!f->dual_split) return RC_E_NOMEM;
  }
  if (!f->fb_halo.empty()) {
    f->fb_split = A.get_n<int64_t>(2 * F);
    if (!f->fb_split) return RC_E_NOMEM;
  }
  f->pidx = A.get_n<int32_t>(P);
  f->pdt = A.get_n<int32_t>(P);
  f->pdm = A.get_n<int32_t>(P);
  f->pc = A.get_n<int32_t>(P);
  if (!f->pidx || !f->pdt || !f->pdm || !f->pc) return RC_E_NOMEM;
  RC_HIP(launch_pair_write(f, mask, s));

  // ---- the records of the wavefront fills, unless the level launches are
  // this family's fill or most budgets take 32-bit cells (then the first
  // solve that needs them builds them)
  f->blk_kind = family_block_kind(f);
  if (f->blk_kind != 0 && 2 * g->M_total <= kMaxBudget && launch_fill_choice(f) < 0) {
    const int er = ensure_records(f, s);
    if (er != RC_OK) return er;
  }
  if (hipStreamSynchronize(s) != hipSuccess) {
    set_last_error_msg("family build: stream synchronisation failed");
    return RC_E_DEVICE;
  }
  return RC_OK;
}

// The block records of the wavefront fills: those of the family's block
// kind, on first use.  Sets has_records and has_wide (false where the family
// is too large for them).  Waits for the stream only where the size of a
// buffer has to be counted: dense records and a bound on the split-panel
// ones need no count.
static int ensure_records(rc_family f, hipStream_t s) {
  if (f->tried_records) return RC_OK;
  Arena& A = f->arena;
  Arena tmp;                       // scratch released on return
  tmp.alloc = A.alloc;
  tmp.free_fn = A.free_fn;
  tmp.user = A.user;
  struct TmpGuard {
    Arena& a;
    hipStream_t s;
    ~TmpGuard() {
      if (a.ptrs.empty()) return;
      (void)hipStreamSynchronize(s);
      a.release_all();
    }
  } guard{tmp, s};
  std::unique_ptr<Staging> up_stage;  // host -> device block starts
  const int64_t F = f->F, P = f->P;
  auto records = [&](int64_t Rn) -> int {
    BlockRecords& R = f->rec;
    const int64_t T3 = f->nblk * kJB * kJB;
    R.src = A.get_n<int32_t>(Rn);
    R.e = A.get_n<int32_t>(Rn * kJB);
    R.kadd = A.get_n<uint32_t>(Rn * kJB);
    R.c = A.get_n<int32_t>(Rn * kJB);
    R.tri_e = A.get_n<int32_t>(T3);
    R.tri_kadd = A.get_n<uint32_t>(T3);
    R.tri_c = A.get_n<int32_t>(T3);
    return R.src && R.e && R.kadd && R.c && R.tri_e && R.tri_kadd && R.tri_c ? RC_OK : RC_E_NOMEM;
  };
  auto read_back = [&](const int64_t* dev, int64_t count, Staging& st) -> int {
    if (!st.data()) return RC_E_NOMEM;
    st.in_flight();
    RC_HIP(hipMemcpyAsync(st.data(), dev, sizeof(int64_t) * (size_t)count, hipMemcpyDeviceToHost,
                          s));
    return sync_landed(st, s);
  };

  if (f->blk_kind == kBlocksFixed && dense_records((F - 1 + kJB - 1) / kJB) <= kMaxRecords) {
    f->nblk = (F - 1 + kJB - 1) / kJB;
    f->bstart = A.get_n<int32_t>(f->nblk + 1);
    f->rec_ptr = A.get_n<int64_t>(f->nblk + 1);
    f->wrec_ptr = A.get_n<int64_t>(f->nblk + 1);
    if (!f->bstart || !f->rec_ptr || !f->wrec_ptr) return RC_E_NOMEM;
    const int ra = records(dense_records(f->nblk));
    if (ra != RC_OK) return ra;
    RC_HIP(launch_blk_dense(f, s));
    f->has_records = true;
    f->wrec_total = P;
  } else {
    std::vector<int32_t> near_h;
    if (f->blk_kind == kBlocksGhost) {
      int32_t* near_d = tmp.get_n<int32_t>(F * kNear);
      Staging st2(sizeof(int32_t) * (size_t)(F * kNear));
      if (!near_d || !st2.data()) return RC_E_NOMEM;
      RC_HIP(launch_near_shifts(f, near_d, s));
      st2.in_flight();
      RC_HIP(hipMemcpyAsync(st2.data(), near_d, sizeof(int32_t) * (size_t)(F * kNear),
                            hipMemcpyDeviceToHost, s));
      const int ss = sync_landed(st2, s);
      if (ss != RC_OK) return ss;
      near_h.assign(st2.at<int32_t>(0), st2.at<int32_t>(0) + F * kNear);
    }
    cut_blocks(f, near_h);
    int64_t* counts = tmp.get_n<int64_t>(F + 1);
    if (!counts) return RC_E_NOMEM;
    const int ub = upload_blocks(f, counts, up_stage, s);
    if (ub != RC_OK) return ub;
    // buffers sized from the bound P when it is small, else from the count
    int64_t rec_cap = std::min<int64_t>(P, f->nblk * F);
    if (f->nblk > 0 && rec_cap > kRecordBound) {
      Staging st3(sizeof(int64_t));
      const int ss = read_back(f->rec_ptr + f->nblk, 1, st3);
      if (ss != RC_OK) return ss;
      rec_cap = *st3.at<int64_t>(0);
    }
    f->has_records = f->nblk > 0 && rec_cap <= kMaxRecords;
    if (f->has_records) {
      const int ra = records(rec_cap);
      if (ra != RC_OK) return ra;
      RC_HIP(launch_blk_fill(f, f->nblk, s));
    }
  }

  // the split-panel fill: one record per (block, source, shift), a block's
  // records sorted in LDS, byte offsets of the table in 31 bits
  if (f->has_records && f->blk_kind == kBlocksFixed) {
    f->has_wide = 2 * f->cells_alloc < INT32_MAX;
    if (!f->wrec_ptr || f->block_pairs > kWMaxRec || P >= ((int64_t)1 << 26)) {
      int64_t* wcounts = tmp.get_n<int64_t>(f->nblk + 1);
      if (!f->wrec_ptr) f->wrec_ptr = A.get_n<int64_t>(f->nblk + 1);
      if (!f->wrec_ptr || !wcounts) return RC_E_NOMEM;
      RC_HIP(launch_wide_count(f, wcounts, s));
      RC_HIP(launch_scan(wcounts, f->wrec_ptr, f->nblk, s));
      Staging st4(sizeof(int64_t) * (size_t)f->nblk);
      const int ss = read_back(wcounts, f->nblk, st4);
      if (ss != RC_OK) return ss;
      f->wrec_total = 0;
      for (int64_t b = 0; b < f->nblk; b++) {
        const int64_t c = st4.at<int64_t>(0)[b];
        f->wrec_total += c;
        f->has_wide = f->has_wide && c <= kWMaxRec;
      }
      f->has_wide = f->has_wide && f->wrec_total < ((int64_t)1 << 26);
    }
  }
  if (up_stage) {
    RC_HIP(hipStreamSynchronize(s));
    up_stage->landed();
  }
  f->tried_records = true;
  return RC_OK;
}

// The shift clusters of the row-push and ghost-zone fills (clu_ptr and their
// number, or a bound on it), on first use.
static int ensure_clusters(rc_family f, hipStream_t s) {
  if (f->clu_ptr) return RC_OK;
  int64_t* counts = f->arena.get_n<int64_t>(f->nblk);
  int64_t* ptr = f->arena.get_n<int64_t>(f->nblk + 1);
  if (!counts || !ptr) return RC_E_NOMEM;
  f->clu_ptr = ptr;
  if (launch_blk_clusters(f, counts, s) != hipSuccess ||
      launch_scan(counts, ptr, f->nblk, s) != hipSuccess) {
    f->clu_ptr = nullptr;
    return RC_E_DEVICE;
  }
  f->clu_total = f->P;                   // every cluster holds a pair
  if (f->P > (int64_t)1 << 14) {
    Staging st(sizeof(int64_t));
    const int e = st.data() ? RC_OK : RC_E_NOMEM;
    if (e != RC_OK) return e;
    st.in_flight();
    RC_HIP(hipMemcpyAsync(st.data(), ptr + f->nblk, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    const int ss = sync_landed(st, s);
    if (ss != RC_OK) return ss;
    f->clu_total = *st.at<int64_t>(0);
  }
  return RC_OK;
}

int rc_build_family(rc_graph g, int32_t mode, int64_t max_sets, void* stream, rc_family* out) {
  if (!g || !out) return RC_E_ARG;
  if (mode != RC_FAMILY_EXACT && mode != RC_FAMILY_PRUNED) return RC_E_ARG;
  if (max_sets < 1) return RC_E_ARG;
  max_sets = std::min<int64_t>(max_sets, kMaxSets);
  rc_family f = new (std::nothrow) rc_family_s();
  if (!f) return RC_E_NOMEM;
  f->g = g;
  f->mode = mode;
  f->arena.alloc = g->arena.alloc;
  f->arena.free_fn = g->arena.free_fn;
  f->arena.user = g->arena.user;
  int st = build_family_impl(f, max_sets, as_stream(stream));
  if (st != RC_OK) {
    (void)hipStreamSynchronize(as_stream(stream));
    f->arena.release_all();
    delete f;
    return st;
  }
  *out = f;
  return RC_OK;
}

int rc_family_stats(rc_family f, rc_family_info* info) {
  if (!f || !info) return RC_E_ARG;
  info->n = f->g->n;
  info->words = f->g->words;
  info->num_sets = f->F;
  info->num_pairs = f->P;
  info->num_levels = (int64_t)f->level_ptr.size() - 1;
  info->table_cells = 0;
  for (int32_t x : f->w_host) info->table_cells += x;
  info->relaxations = f->relax;
  info->T_total = f->g->T_total;
  info->M_total = f->g->M_total;
  info->max_row = f->max_row;
  return RC_OK;
}

int rc_min_budget(rc_family f, void* stream, int64_t* B_min) {
  if (!f || !B_min) return RC_E_ARG;
  const int64_t hi0 = 2 * f->g->M_total;           // the chain {V} peaks at 2 M(V)
  if (hi0 >= INT32_MAX) return RC_E_OVERFLOW;
  hipStream_t s = as_stream(stream);
  if (!f->bmin_scratch) {
    f->bmin_scratch = f->arena.get(min_budget_scratch_bytes(f, (int32_t)hi0));
    if (!f->bmin_scratch) return RC_E_NOMEM;
  }
  Staging stage(sizeof(int64_t));
  stage.in_flight();
  int64_t* out = stage.data() ? stage.at<int64_t>(0) : nullptr;
  RC_HIP(launch_min_budget(f, (int32_t)hi0, f->bmin_scratch, &out, s));
  int64_t found = 0;                       // no pinned memory: out is on the device
  if (!stage.data())
    RC_HIP(hipMemcpyAsync(&found, out, sizeof(found), hipMemcpyDeviceToHost, s));
  const int ss = sync_landed(stage, s);
  if (ss != RC_OK) return ss;
  *B_min = stage.data() ? *out : found;
  return RC_OK;
}

int rc_solve_dual(rc_family f, int64_t B, int32_t objective, void* stream, int64_t* t_opt,
                  int64_t* m_opt, float* fill_ms, int32_t* k, int32_t* chain_host,
                  int32_t* seg_host, uint8_t* cached_host, int64_t* overhead, int64_t* peak,
                  int64_t* cache_mem) {
  DualBuffers need;
  const int st0 = dual_buffers(f, B, objective, &need);
  if (st0 != RC_OK) return st0;
  hipStream_t s = as_stream(stream);
  rcdp::Arena A;
  A.alloc = f->arena.alloc;
  A.free_fn = f->arena.free_fn;
  A.user = f->arena.user;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  auto finish = [&](int st) {
    (void)hipStreamSynchronize(s);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    A.release_all();
    return st;
  };
  DualBuffers buf = need;
  buf.D = A.get_n<uint32_t>(need.cells);
  buf.st = A.get_n<DevStatus>(1);
  buf.chain = A.get_n<int32_t>(f->F);
  const int64_t n = f->g->n, kmax = std::min<int64_t>(f->F, n + 1);
  StageLayout lay;
  const size_t o_st = lay.add<DevStatus>(2), o_ch = lay.add<int32_t>(kmax),
               o_sg = lay.add<int32_t>(n), o_ca = lay.add<uint8_t>(n);
  Staging stage(lay.bytes);
  if (!buf.D || !buf.st || !buf.chain || !stage.data()) return finish(RC_E_NOMEM);
  buf.host = &stage;
  buf.host_st = stage.at<DevStatus>(o_st);
  buf.out_chain = stage.at<int32_t>(o_ch);
  buf.seg = stage.at<int32_t>(o_sg);
  buf.cached = stage.at<uint8_t>(o_ca);
  if (fill_ms && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess))
    return finish(RC_E_DEVICE);
  const int st = dual_solve(f, objective, buf, e0, e1, s, t_opt, m_opt, k, chain_host, seg_host,
                            cached_host, overhead, peak, cache_mem);
  if (fill_ms && st >= 0) {
    float ms = -1.f;
    if (hipEventElapsedTime(&ms, e0, e1) != hipSuccess) ms = -1.f;
    *fill_ms = ms;
  }
  return finish(st);
}

int rc_family_sets(rc_family f, uint64_t* bits_host, void* stream) {
  if (!f || !bits_host) return RC_E_ARG;
  const int words = f->g->words;
  hipStream_t s = as_stream(stream);
  std::vector<uint64_t> wm((size_t)words * f->fstride);
  if (!wm.empty())
    RC_HIP(hipMemcpyAsync(wm.data(), f->bits, sizeof(uint64_t) * wm.size(),
                          hipMemcpyDeviceToHost, s));
  RC_HIP(hipStreamSynchronize(s));
  for (int64_t i = 0; i < f->F; i++)
    for (int w = 0; w < words; w++) bits_host[i * words + w] = wm[(size_t)w * f->fstride + i];
  return RC_OK;
}

void rc_family_free(rc_family f) {
  if (!f) return;
  (void)hipDeviceSynchronize();
  f->arena.release_all();
  delete f;
}

// ------------------------------------------------------------------ solve

static void destroy_events(rc_solution sol) {
  for (hipEvent_t* e : {&sol->ev0, &sol->ev1, &sol->evk0, &sol->evk1})
    if (*e) {
      (void)hipEventDestroy(*e);
      *e = nullptr;
    }
}

// The cheapest fill of a family by measured costs on this GPU: 0 the level
// launches, 5 the block launches, 3 the family's wavefront.  The wavefront
// runs its 256-cell columns at most three (the split-panel fill: four) per
// compute unit at a time, each through every row of the table at about 2.5 us
// per row (2 us where only a few columns run).  A level launch costs about
// 3.5 us, plus the source reads of its pairs (2 bytes per relaxation) at about
// 6 TB/s, partly beside each other; a block launch of 16 rows about 9.5 us,
// 27 ns per cell of its halo and the same reads.  Few levels of many sets or of
// very long rows take the level launches, many levels of short rows the
// blocks, of long ones the wavefront.  Whole fills in ms, level / block / the
// wavefront that the family takes, its records included: densenet121_t10 2.27
// / 0.30 / 0.94, resnet50_t10 0.68 / 0.13 / 0.35, a 16-node chain 0.065 /
// 0.017 / 0.061, layered24 0.097 / 0.094 / 0.12, ladder40 0.18 / 0.35 / 0.55,
// U-Net 0.45 / - / 0.68, ResNet-50 0.88 / - / 0.66, DenseNet-121 4.1 / - /
// 1.8.
static int cheapest_fill(rc_family f) {
  const int64_t levels = (int64_t)f->level_ptr.size() - 1;
  const int64_t slots = (f->blk_kind == kBlocksGhost ? 3 : wide_slots_per_cu(3)) *
                        (int64_t)num_cus();
  const int64_t col_rounds = ((f->max_row + kWC - 1) / kWC + slots - 1) / slots;
  const double reads = 2.0 * (double)f->relax / 6.0e6;
  const double wave_us = 2.5 * (double)f->F * (double)col_rounds;
  const double level_us = 3.5 * (double)levels + reads;
  double block_us = reads;
  for (int32_t h : f->fb_halo) block_us += 9.5 + 0.027 * (double)h;
  if (!f->fb_halo.empty() && block_us < wave_us && block_us < level_us) return 5;
  return level_us < wave_us ? 0 : 3;
}

static bool forces_wavefront(const char* env) {
  return env && (std::strcmp(env, "wavefront") == 0 || std::strcmp(env, "wide") == 0 ||
                 std::strcmp(env, "ghost") == 0);
}

// The fill without records (0 or 5) that a solve of the family takes now, or
// -1: a wavefront.
static int launch_fill_choice(rc_family f) {
  const char* env = std::getenv("RCDP_FILL");
  if (env && std::strcmp(env, "level") == 0) return 0;
  if (env && std::strcmp(env, "block") == 0) return f->fb_halo.empty() ? 0 : 5;
  if (forces_wavefront(env)) return -1;
  const int c = cheapest_fill(f);
  return c == 3 ? -1 : c;
}

// The fill of a solve (rc_solution_fill_path's numbers), with the records it
// reads built.
static int choose_fill_path(rc_family f, hipStream_t s, int32_t* path) {
  *path = 0;
  if (f->blk_kind == 0) return RC_OK;
  const int launches = launch_fill_choice(f);
  if (launches >= 0) {
    *path = launches;
    return RC_OK;
  }
  const int er = ensure_records(f, s);
  if (er != RC_OK) return er;
  if (!f->has_records) return RC_OK;
  // the family's wavefront fill: ghost-zone blocks, or fixed blocks of kJB
  // with the split-panel fill when it can take the family
  const int wave = f->blk_kind == kBlocksGhost ? 2 : (f->has_wide ? 3 : 1);
  const char* env = std::getenv("RCDP_FILL");
  if (env && std::strcmp(env, "wavefront") == 0 && f->blk_kind == kBlocksFixed)
    *path = 1;
  else if (env && (std::strcmp(env, "wide") == 0 || std::strcmp(env, "ghost") == 0))
    *path = wave;
  else
    *path = wave == 1 ? 0 : wave;
  return *path == 1 || *path == 2 ? ensure_clusters(f, s) : RC_OK;
}

}  // extern "C"

// A solution handle with its buffers and events.  Nothing of the solve is
// enqueued yet, but the family's records are where this is the first solve
// that reads them: on an error s has been waited for, so that a later solve,
// on whatever stream, finds them written.
static int new_solution(rc_family f, int64_t B, int32_t objective, hipStream_t s,
                        rc_solution* out) {
  if (!f || B < 0) return RC_E_ARG;
  if (objective != RC_TIME_CENTRIC && objective != RC_MEMORY_CENTRIC) return RC_E_ARG;
  const int64_t Beff = std::min<int64_t>(B, 2 * f->g->M_total);
  if (Beff > kMaxBudget32) return RC_E_OVERFLOW;
  // a budget beyond the 16-bit cells: 32-bit cells and the level fill
  const bool cell32 = Beff > kMaxBudget;
  rc_solution sol = new (std::nothrow) rc_solution_s();
  if (!sol) return RC_E_NOMEM;
  sol->f = f;
  sol->B = B;
  sol->Beff = Beff;
  sol->objective = objective;
  sol->arena.alloc = f->arena.alloc;
  sol->arena.free_fn = f->arena.free_fn;
  sol->arena.user = f->arena.user;
  auto fail = [&](int st) {
    (void)hipStreamSynchronize(s);           // the family's records may be on their way
    destroy_events(sol);
    sol->arena.release_all();
    delete sol;
    return st;
  };
  sol->cell32 = cell32;
  if (cell32)
    sol->m32 = sol->arena.get_n<uint32_t>(f->cells_alloc);
  else
    sol->m = sol->arena.get_n<uint16_t>(f->cells_alloc);
  sol->status = sol->arena.get_n<DevStatus>(1);
  sol->chain = sol->arena.get_n<int32_t>(f->F);
  if (!(sol->m || sol->m32) || !sol->status || !sol->chain) return fail(RC_E_NOMEM);
  if (hipEventCreate(&sol->ev0) != hipSuccess || hipEventCreate(&sol->ev1) != hipSuccess)
    return fail(RC_E_DEVICE);
  if (!cell32) {
    const int cp = choose_fill_path(f, s, &sol->fill_path);
    if (cp != RC_OK) return fail(cp);
  }
  if (sol->fill_path != 0 && sol->fill_path != 5 &&
      (hipEventCreate(&sol->evk0) != hipSuccess || hipEventCreate(&sol->evk1) != hipSuccess))
    return fail(RC_E_DEVICE);
  if (sol->fill_path == 3) {
    sol->wslab = static_cast<char*>(sol->arena.get(wide_slab_bytes(f)));
    if (!sol->wslab) return fail(RC_E_NOMEM);
  } else if (sol->fill_path == 1 || sol->fill_path == 2) {
    const int64_t K = sol->fill_path == 2 ? ghost_columns(f) : blocked_columns(f);
    sol->progress = sol->arena.get_n<int32_t>(K);
    sol->ticket = sol->arena.get_n<int32_t>(1);
    sol->crec = sol->arena.get_n<int32_t>(f->clu_total * kRecInts);
    sol->crec_tmp = sol->arena.get_n<int32_t>(f->clu_total * kRecInts);
    sol->live_cap = (int32_t)std::min<int64_t>(K, kLiveCap);
    sol->live = sol->arena.get_n<int32_t>(f->nblk * sol->live_cap * 2);
    sol->blk_meta = sol->arena.get_n<int32_t>(f->nblk * kMetaInts);
    if (sol->fill_path == 2)
      sol->tri = sol->arena.get_n<int32_t>(f->nblk * kJB * kTriInts);
    else
      sol->push = sol->arena.get_n<int32_t>(f->nblk * kJB * kPushInts);
    sol->sentinel = sol->arena.get_n<uint16_t>(8);
    if (!sol->progress || !sol->ticket || !sol->crec || !sol->crec_tmp || !sol->live ||
        !sol->blk_meta || !(sol->push || sol->tri) || !sol->sentinel)
      return fail(RC_E_NOMEM);
  }
  *out = sol;
  return RC_OK;
}

static void drop_solution(rc_solution sol) {
  destroy_events(sol);
  sol->arena.release_all();
  delete sol;
}

// The selection result read back from the device, into the handle.
static int settle_solution(rc_solution sol, const DevStatus& hs, float fill_ms, float kernel_ms) {
  if (hs.error) {
    set_last_error_msg(hs.error == 3   ? "wavefront fill: a wait timed out (kernel aborted)"
                       : hs.error == 4 ? "ghost fill: an in-block shift exceeds the halo"
                                       : "DP fill kernel reported an inconsistency");
    return RC_E_DEVICE;
  }
  sol->fill_ms = fill_ms;
  sol->kernel_ms = kernel_ms;
  sol->t_star = hs.t_sel;
  sol->m_star = hs.t_sel >= 0 ? hs.m_sel : -1;
  sol->result = hs.t_sel >= 0 ? RC_OK : RC_INFEASIBLE;
  return sol->result;
}

static float elapsed(hipEvent_t a, hipEvent_t b) {
  float ms = -1.f;
  if (!a || !b || hipEventElapsedTime(&ms, a, b) != hipSuccess) return -1.f;
  return ms;
}

// Status of a launcher that failed: it reports the family's allocator
// returning NULL as hipErrorOutOfMemory.
static int launch_status(const char* what, hipError_t e) {
  if (e == hipErrorOutOfMemory) return RC_E_NOMEM;
  set_last_error(what, e);
  return RC_E_DEVICE;
}

// rc_solve and rc_solve_dominance: one table fill, then the selection of t*.
static int solve_one(rc_family f, int64_t B, int32_t objective, void* stream, rc_solution* out,
                     int64_t* t_opt, int64_t* m_opt, bool dominance) {
  if (!f || !out) return RC_E_ARG;
  hipStream_t s = as_stream(stream);
  rc_solution sol = nullptr;
  const int st0 = new_solution(f, B, objective, s, &sol);
  if (st0 != RC_OK) return st0;
  if (dominance && sol->cell32) {      // the weak-front kernels take 16-bit cells only
    drop_solution(sol);
    return RC_E_OVERFLOW;
  }
  auto fail = [&](int st) {
    (void)hipStreamSynchronize(s);
    drop_solution(sol);
    return st;
  };
  if (hipEventRecord(sol->ev0, s) != hipSuccess) return fail(RC_E_DEVICE);
  if (launch_solve_init(&sol, 1, s) != hipSuccess) return fail(RC_E_DEVICE);
  hipError_t fe = sol->fill_path == 5   ? launch_fill_block(&sol, 1, s)
                  : sol->fill_path == 3 ? launch_fill_wide(sol, s)
                  : sol->fill_path == 2 ? launch_fill_ghost(sol, s)
                  : sol->fill_path == 1 ? launch_fill_blocked(sol, s)
                                        : launch_fill(sol, s);
  if (fe == hipSuccess && dominance) fe = launch_fronts(sol, s);
  if (fe != hipSuccess)
    return fail(launch_status(sol->fill_path == 5   ? "block fill launch"
                              : sol->fill_path == 3 ? "split-panel fill launch"
                              : sol->fill_path == 2 ? "ghost fill launch"
                              : sol->fill_path == 1 ? "blocked fill launch"
                                                    : "level fill launch",
                              fe));
  if (hipEventRecord(sol->ev1, s) != hipSuccess) return fail(RC_E_DEVICE);
  Staging stage(sizeof(DevStatus));
  if (!stage.data()) return fail(RC_E_NOMEM);
  stage.in_flight();
  if (launch_select(&sol, 1, stage.at<DevStatus>(0), s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return fail(RC_E_DEVICE);
  stage.landed();
  const DevStatus hs = *stage.at<DevStatus>(0);
  const float fill_ms = elapsed(sol->ev0, sol->ev1);
  const float kernel_ms = sol->evk0 ? elapsed(sol->evk0, sol->evk1) : fill_ms;
  const int st = settle_solution(sol, hs, fill_ms, kernel_ms);
  if (st < 0) return fail(st);
  if (t_opt) *t_opt = sol->t_star;
  if (m_opt) *m_opt = sol->m_star;
  *out = sol;
  return st;
}

extern "C" {

int rc_solve(rc_family f, int64_t B, int32_t objective, void* stream, rc_solution* out,
             int64_t* t_opt, int64_t* m_opt) {
  return solve_one(f, B, objective, stream, out, t_opt, m_opt, false);
}

int rc_solve_dominance(rc_family f, int64_t B, void* stream, rc_solution* out, int64_t* t_opt,
                       int64_t* m_opt) {
  return solve_one(f, B, RC_TIME_CENTRIC, stream, out, t_opt, m_opt, true);
}

int rc_solve_batch(rc_family f, const int64_t* B_host, int32_t nb, int32_t objective,
                   void* stream, rc_solution* out_host, int64_t* t_opt, int64_t* m_opt) {
  if (!f || !B_host || !out_host || nb <= 0) return RC_E_ARG;
  hipStream_t s = as_stream(stream);
  std::vector<rc_solution> sols;
  auto fail = [&](int st) {
    (void)hipStreamSynchronize(s);
    for (rc_solution x : sols) drop_solution(x);
    return st;
  };
  for (int32_t b = 0; b < nb; b++) {
    rc_solution x = nullptr;
    const int st = new_solution(f, B_host[b], objective, s, &x);
    if (st != RC_OK) return fail(st);
    sols.push_back(x);
  }
  rc_solution s0 = sols[0];
  if (hipEventRecord(s0->ev0, s) != hipSuccess) return fail(RC_E_DEVICE);
  if (launch_solve_init(sols.data(), nb, s) != hipSuccess) return fail(RC_E_DEVICE);
  std::vector<BParams> host_prm;
  std::vector<GParams> host_gprm;
  std::vector<WParams> host_wprm;
  // one batched launch when every table takes the same fill (budgets beyond
  // the 16-bit cells take the level fill, one table at a time)
  bool same = true;
  for (rc_solution x : sols) same = same && x->fill_path == s0->fill_path;
  if (!same) {
    for (rc_solution x : sols) {
      const hipError_t fe = x->fill_path == 5   ? launch_fill_block(&x, 1, s)
                            : x->fill_path == 3 ? launch_fill_wide(x, s)
                            : x->fill_path == 2 ? launch_fill_ghost(x, s)
                            : x->fill_path == 1 ? launch_fill_blocked(x, s)
                                                : launch_fill(x, s);
      if (fe != hipSuccess) return fail(launch_status("fill launch", fe));
    }
  } else if (s0->fill_path == 5) {
    const hipError_t fe = launch_fill_block(sols.data(), nb, s);
    if (fe != hipSuccess) return fail(launch_status("batched block fill launch", fe));
  } else if (s0->fill_path == 3) {
    host_wprm.resize((size_t)nb);
    WParams* dev_prm = s0->arena.get_n<WParams>(nb);
    if (!dev_prm) return fail(RC_E_NOMEM);
    const hipError_t fe = launch_fill_wide_batch(sols.data(), nb, host_wprm.data(), dev_prm, s);
    if (fe != hipSuccess) return fail(launch_status("batched split-panel fill launch", fe));
  } else if (s0->fill_path == 2) {
    host_gprm.resize((size_t)nb);
    GParams* dev_prm = s0->arena.get_n<GParams>(nb);
    if (!dev_prm) return fail(RC_E_NOMEM);
    const hipError_t fe = launch_fill_ghost_batch(sols.data(), nb, host_gprm.data(), dev_prm, s);
    if (fe != hipSuccess) return fail(launch_status("batched ghost fill launch", fe));
  } else if (s0->fill_path == 1) {
    host_prm.resize((size_t)nb);
    BParams* dev_prm = s0->arena.get_n<BParams>(nb);
    if (!dev_prm) return fail(RC_E_NOMEM);
    const hipError_t fe = launch_fill_blocked_batch(sols.data(), nb, host_prm.data(), dev_prm, s);
    if (fe != hipSuccess) return fail(launch_status("batched blocked fill launch", fe));
  } else {
    for (rc_solution x : sols) {
      const hipError_t fe = launch_fill(x, s);
      if (fe != hipSuccess) return fail(launch_status("level fill launch", fe));
    }
  }
  if (hipEventRecord(s0->ev1, s) != hipSuccess) return fail(RC_E_DEVICE);
  Staging stage(sizeof(DevStatus) * (size_t)nb);
  if (!stage.data()) return fail(RC_E_NOMEM);
  stage.in_flight();
  if (launch_select(sols.data(), nb, stage.at<DevStatus>(0), s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return fail(RC_E_DEVICE);
  stage.landed();
  const float fill_ms = elapsed(s0->ev0, s0->ev1);
  const float kernel_ms = s0->evk0 ? elapsed(s0->evk0, s0->evk1) : fill_ms;
  for (int32_t b = 0; b < nb; b++) {
    const int st = settle_solution(sols[b], stage.at<DevStatus>(0)[b], fill_ms, kernel_ms);
    if (st < 0) return fail(st);
  }
  for (int32_t b = 0; b < nb; b++) {
    out_host[b] = sols[b];
    if (t_opt) t_opt[b] = sols[b]->t_star;
    if (m_opt) m_opt[b] = sols[b]->m_star;
  }
  return RC_OK;
}

int rc_solution_fill_ms(rc_solution s, float* ms) {
  if (!s || !ms) return RC_E_ARG;
  *ms = s->fill_ms;
  return RC_OK;
}

int rc_solution_fill_kernel_ms(rc_solution s, float* ms) {
  if (!s || !ms) return RC_E_ARG;
  *ms = s->kernel_ms;
  return RC_OK;
}

int rc_solution_fill_path(rc_solution s, int32_t* path) {
  if (!s || !path) return RC_E_ARG;
  *path = s->fill_path == 0 && s->cell32 ? 4 : s->fill_path;
  return RC_OK;
}

int rc_solution_trace_path(rc_solution s, int32_t* path) {
  if (!s || !path) return RC_E_ARG;
  *path = s->trace_path;
  return RC_OK;
}

int rc_reconstruct(rc_solution sol, void* stream, int32_t* k, int32_t* chain_host,
                   int32_t* seg_host, uint8_t* cached_host, int64_t* overhead, int64_t* peak,
                   int64_t* cache_mem) {
  if (!sol) return RC_E_ARG;
  if (sol->result != RC_OK) return RC_INFEASIBLE;
  hipStream_t s = as_stream(stream);
  rc_family f = sol->f;
  const int n = f->g->n;
  // the chain has at most min(F, n + 1) sets: every step adds a node
  const int64_t kmax = std::min<int64_t>(f->F, (int64_t)n + 1);
  StageLayout lay;
  const size_t o_st = lay.add<DevStatus>(1), o_ch = lay.add<int32_t>(kmax),
               o_sg = lay.add<int32_t>(n), o_ca = lay.add<uint8_t>(n);
  Staging stage(lay.bytes);
  if (!stage.data()) return RC_E_NOMEM;
  const ScheduleOut sched{stage.at<int32_t>(o_ch), stage.at<int32_t>(o_sg),
                          stage.at<uint8_t>(o_ca), stage.at<DevStatus>(o_st)};
  stage.in_flight();
  const hipError_t te = launch_trace(sol, sched, s);
  if (te == hipErrorOutOfMemory) {
    stage.landed();
    return RC_E_NOMEM;
  }
  if (te != hipSuccess) {
    set_last_error("traceback launch", te);
    return RC_E_DEVICE;
  }
  RC_HIP(hipStreamSynchronize(s));
  stage.landed();
  const DevStatus hs = *stage.at<DevStatus>(o_st);
  if (hs.error || hs.k < 0 || hs.k > kmax) {
    set_last_error_msg("traceback: optarg walk did not end at (empty set, 0)");
    return RC_E_DEVICE;
  }
  if (k) *k = hs.k;
  if (chain_host) std::copy(stage.at<int32_t>(o_ch), stage.at<int32_t>(o_ch) + hs.k, chain_host);
  if (seg_host) std::copy(stage.at<int32_t>(o_sg), stage.at<int32_t>(o_sg) + n, seg_host);
  if (cached_host) std::copy(stage.at<uint8_t>(o_ca), stage.at<uint8_t>(o_ca) + n, cached_host);
  if (overhead) *overhead = hs.overhead;
  if (peak) *peak = hs.peak;
  if (cache_mem) *cache_mem = hs.cache_mem;
  return RC_OK;
}

int rc_export_table(rc_solution sol, int64_t first, int64_t count, int64_t* m_host,
                    int32_t* arg_host, void* stream) {
  if (!sol || first < 0 || count < 0 || first + count > sol->f->F) return RC_E_ARG;
  rc_family f = sol->f;
  hipStream_t s = as_stream(stream);
  const int64_t W = f->g->T_total + 1;
  if (arg_host && !sol->arg) {               // optarg of the whole table, derived once
    sol->arg = sol->arena.get_n<uint16_t>(f->cells_alloc);
    if (!sol->arg) return RC_E_NOMEM;
    RC_HIP(launch_arg_all(sol, s));
  }
  const int64_t c0 = f->row_off_host[first], c1 = f->row_off_host[first + count];
  std::vector<uint16_t> mm(sol->cell32 ? 0 : c1 - c0), aa(arg_host ? c1 - c0 : 0);
  std::vector<uint32_t> mm32(sol->cell32 ? c1 - c0 : 0);
  if (c1 > c0) {
    if (sol->cell32)
      RC_HIP(hipMemcpyAsync(mm32.data(), sol->m32 + c0, 4 * (c1 - c0), hipMemcpyDeviceToHost, s));
    else
      RC_HIP(hipMemcpyAsync(mm.data(), sol->m + c0, 2 * (c1 - c0), hipMemcpyDeviceToHost, s));
    if (arg_host)
      RC_HIP(hipMemcpyAsync(aa.data(), sol->arg + c0, 2 * (c1 - c0), hipMemcpyDeviceToHost, s));
  }
  RC_HIP(hipStreamSynchronize(s));
  const uint32_t inf = sol->cell32 ? 0xFFFFFFFFu : kInfM;
  for (int64_t r = 0; r < count; r++) {
    const int64_t set = first + r;
    const int64_t off = f->row_off_host[set] - c0;
    const int64_t w = f->w_host[set];
    for (int64_t t = 0; t < W; t++) {
      const bool in = t < w;
      const uint32_t mv = !in ? inf : sol->cell32 ? mm32[off + t] : mm[off + t];
      const uint32_t av = (in && arg_host) ? aa[off + t] : kNoArg;
      if (m_host) m_host[r * W + t] = mv == inf ? -1 : (int64_t)mv;
      if (arg_host) arg_host[r * W + t] = (mv == inf || av == kNoArg) ? -1 : (int32_t)av;
    }
  }
  return RC_OK;
}

void rc_solution_free(rc_solution sol) {
  if (!sol) return;
  (void)hipDeviceSynchronize();
  destroy_events(sol);
  sol->arena.release_all();
  delete sol;
}

}  // extern "C"
