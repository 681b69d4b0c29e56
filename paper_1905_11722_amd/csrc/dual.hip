// Memory-indexed form of Algorithm 1's recursion (Section 4.2, Appendix A).
//
// Algorithm 1 walks states (L, t, m) -- a chain ending at lower set L with
// forward time t and cached memory m -- and keeps, per (L, t), the least m.
// A pair L < L' moves (L, t, m) to (L', t + dt, m + dm) when m + c <= B; the
// test depends on m alone.  This table keeps, per (L, m), the least t (time
// centric) or the greatest t (memory centric, Section 4.4) instead: a later
// step adds the same time to two states of equal memory, so the kept one is
// never worse, and the optimum over row V is Algorithm 1's t* with
// opt[V, t*] = the least m that attains it.  Rows span m in [0, W),
// W = min(B, M(V)) + 1 (every cached memory is M(U) for a node set U), so the
// budget test becomes a window on the source index: target cell m' reads
// source cell m' - dm when 0 <= m' - dm <= B - c.
//
// Layout: D[L * W + m], uint32.  Time centric: t, kDualNone (the largest
// value) where no chain reaches (L, m); memory centric: t + 1, 0 where none
// does, so that both combine with one atomic min / max.
// Two fills.  Where a family has many small levels, one launch per block of
// consecutive targets (k_dual_block); else one launch per group of equal-size
// sets (k_dual_level: sets of equal size never contain each other).  In the
// latter, block (x, y, z) is 256 cells of target y of the group and the z-th
// run of kDualPairs of its pairs (read through wave-uniform scalar loads); a
// thread issues the source loads of kDualBatch pairs together and folds its
// candidate into the target cell with one atomic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "rc_internal.h"
#include "dual.h"
#include "schedule.h"

namespace rcdp {

namespace {

constexpr int kDualThreads = 256;
constexpr int kDualPairs = 4;                       // pairs per block
constexpr int kDualBatch = 4;                       // source loads in flight per thread
constexpr uint32_t kDualNone = 0xFFFFFFFFu;

__global__ void k_dual_init(uint32_t* D, int64_t cells, int tc, DevStatus* st) {
  for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < cells;
       x += (int64_t)gridDim.x * blockDim.x)
    D[x] = x == 0 ? (tc ? 0u : 1u) : (tc ? kDualNone : 0u);   // (empty set, m = 0): t = 0
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->error = 0;
    st->t_sel = -1;
    st->m_sel = -1;
  }
}

template <bool kTC>
__global__ __launch_bounds__(kDualThreads) void k_dual_level(
    int64_t lb, int32_t W, int32_t B, const int64_t* __restrict__ pred_ptr,
    const int32_t* __restrict__ pidx, const int32_t* __restrict__ pdt,
    const int32_t* __restrict__ pdm, const int32_t* __restrict__ pc, uint32_t* __restrict__ D) {
  constexpr uint32_t kNone = kTC ? kDualNone : 0u;
  const int64_t j = lb + blockIdx.y;
  const int32_t mp = blockIdx.x * kDualThreads + threadIdx.x;
  const int64_t q0 = pred_ptr[j], q1 = pred_ptr[j + 1];
  const int64_t p0 = q0 + (int64_t)blockIdx.z * kDualPairs;
  const int64_t p1 = min(q1, p0 + kDualPairs);
  if (mp >= W || p0 >= p1) return;
  uint32_t acc = kNone;
  for (int64_t pb = p0; pb < p1; pb += kDualBatch) {
    uint32_t x[kDualBatch];
    int32_t dt[kDualBatch];
#pragma unroll
    for (int k = 0; k < kDualBatch; k++) {
      // every load is issued (a pair past the run re-reads the run's first
      // one, a cell outside the window reads cell 0) and tested afterwards
      const int64_t p = pb + k < p1 ? pb + k : p0;
      const int32_t m = mp - pdm[p];                 // source cell: memory before the step
      const bool ok = pb + k < p1 && m >= 0 && m <= B - pc[p];   // m + c <= B (Algorithm 1)
      const uint32_t v = D[(int64_t)pidx[p] * W + (ok ? m : 0)];
      x[k] = ok ? v : kNone;
      dt[k] = pdt[p];
    }
#pragma unroll
    for (int k = 0; k < kDualBatch; k++) {
      if (x[k] == kNone) continue;
      const uint32_t y = x[k] + (uint32_t)dt[k];
      acc = kTC ? min(acc, y) : max(acc, y);
    }
  }
  if (acc == kNone) return;
  if (kTC)
    atomicMin(&D[j * (int64_t)W + mp], acc);
  else
    atomicMax(&D[j * (int64_t)W + mp], acc);
}

// One launch per block of 8 or 4 consecutive targets.  Launch b has
// two kinds of workgroups, beside each other:
//  - panel (block b + 1): the pairs from sources before block b, which are
//    final, folded into the rows of block b + 1 with atomics as above;
//  - rows (block b): for kDualOwn cells, the rows start from their panel (the
//    launch before), take the pairs from the previous block's rows, then
//    finish one after the other, each relaxing the later rows of the block.
// A step reads cells to its left only (m - dm), so a rows workgroup
// recomputes the `halo` cells left of its own, which no exchange with another
// workgroup is needed for: along a path of pairs inside the block the
// additions sum to at most M(L_last) - M(L_first), because
// dm = M(bd(L') \ L) <= M(L' \ L), and the host passes the largest such
// difference.  Halo cells belong to another workgroup that stores them final
// meanwhile; reading either value gives the same minimum.
//
// Rows workgroup: 8 slots of 128 threads, a slot a target, a thread up to
// kDualK cells 128 apart, in registers; finished rows lie in LDS.  One
// barrier per row.  Bound by a launch's chain of cold loads (offsets, pairs,
// cells) and the rows' steps, about 8 us a block, up to 13 with the widest
// halos and panels: DenseNet-121 (426 rows of 4097 cells, 54 blocks) 0.55 ms
// against 1.51 with a launch per level, ResNet-50 0.21 against 0.53.
// Measured: 256 own cells 0.61 ms, 64 0.55; runs of 8 or 32 pairs 0.64 and
// 0.57 (16: 0.55).
constexpr int kDualOwn = 128;
constexpr int kDualSlots = 8;
constexpr int kDualLanes = 128;
constexpr int kDualK = 10;
constexpr int kDualSpan = kDualLanes * kDualK;
constexpr int kDualHalo = kDualSpan - kDualOwn;
constexpr int kDualRun = 16;                        // pairs per panel item

struct DualBlock {
  int64_t j0, j1;             // rows of the block (none: j0 == j1)
  int64_t n0, n1;             // rows of the next block
  int32_t halo, row_blocks;   // rows workgroups
  int32_t tiles, runs;        // panel items: targets x tiles of 256 cells x runs of pairs
};

template <bool kTC>
__device__ __forceinline__ uint32_t dual_better(uint32_t a, uint32_t b) {
  return kTC ? min(a, b) : max(a, b);
}

template <bool kTC>
__global__ __launch_bounds__(kDualSlots* kDualLanes) void k_dual_block(
    DualBlock g, int32_t W, int32_t B, const int64_t* __restrict__ pred_ptr,
    const int64_t* __restrict__ split, const int32_t* __restrict__ pidx,
    const int32_t* __restrict__ pdt, const int32_t* __restrict__ pdm,
    const int32_t* __restrict__ pc, uint32_t* D) {
  constexpr uint32_t kNone = kTC ? kDualNone : 0u;
  __shared__ uint32_t s_row[kDualSlots][kDualSpan];
  __shared__ int4 s_tri[kDualSlots][kDualSlots];      // [target][source] dm, dt, B - c (-1: none)
  const int tid = threadIdx.x;
  if ((int32_t)blockIdx.x >= g.row_blocks) {
    // ---- panel of the next block: four items of 256 threads
    const int32_t item = __builtin_amdgcn_readfirstlane(
        ((int32_t)blockIdx.x - g.row_blocks) * 4 + tid / 256);
    const int32_t per = g.tiles * g.runs;
    const int64_t j = g.n0 + item / per;
    if (j >= g.n1) return;
    const int32_t rest = item % per;
    const int32_t mp = (rest % g.tiles) * 256 + (tid & 255);
    const int64_t p0 = pred_ptr[j] + (int64_t)(rest / g.tiles) * kDualRun;
    const int64_t p1 = split[2 * j];
    if (p0 >= p1) return;
    // lane q holds the q-th pair of the run (past its end: none passes)
    const int lane = tid & 63;
    int32_t src = 0, dmv = 0, dtv = 0, tau = -1;
    if (lane < kDualRun && p0 + lane < p1) {
      src = pidx[p0 + lane];
      dmv = pdm[p0 + lane];
      dtv = pdt[p0 + lane];
      tau = B - pc[p0 + lane];
    }
    uint32_t x[kDualRun];
#pragma unroll
    for (int k = 0; k < kDualRun; k++) {
      const int32_t m = mp - __builtin_amdgcn_readlane(dmv, k);
      const int32_t tk = __builtin_amdgcn_readlane(tau, k);
      const bool ok = mp < W && m >= 0 && m <= tk;
      const uint32_t v = D[(int64_t)__builtin_amdgcn_readlane(src, k) * W + (ok ? m : 0)];
      x[k] = ok ? v : kNone;
    }
    uint32_t acc = kNone;
#pragma unroll
    for (int k = 0; k < kDualRun; k++)
      if (x[k] != kNone)
        acc = dual_better<kTC>(acc, x[k] + (uint32_t)__builtin_amdgcn_readlane(dtv, k));
    if (acc == kNone) return;
    if (kTC)
      atomicMin(&D[j * (int64_t)W + mp], acc);
    else
      atomicMax(&D[j * (int64_t)W + mp], acc);
    return;
  }
  // ---- rows of the block
  const int slot = __builtin_amdgcn_readfirstlane(tid / kDualLanes);
  const int l128 = tid % kDualLanes, lane = tid & 63;
  const int nrows = (int)(g.j1 - g.j0);
  const int64_t j = g.j0 + slot;
  const int32_t m0 = (int32_t)blockIdx.x * kDualOwn;
  const int32_t mb = max(0, m0 - g.halo);                 // first cell computed
  const int32_t cells = min(W, m0 + kDualOwn) - mb;       // at most kDualSpan
  if (tid < kDualSlots * kDualSlots) s_tri[tid / kDualSlots][tid % kDualSlots].z = -1;
  uint32_t acc[kDualK];
#pragma unroll
  for (int k = 0; k < kDualK; k++) acc[k] = kNone;
  __syncthreads();
  if (slot < nrows) {
    const int64_t p1 = split[2 * j], p2 = split[2 * j + 1], p3 = pred_ptr[j + 1];
    // lane q: the q-th pair from the previous block's rows, and from the block's
    int32_t csrc = 0, cdm = 0, cdt = 0, ctau = -1;
    if (lane < (int)(p2 - p1)) {
      csrc = pidx[p1 + lane];
      cdm = pdm[p1 + lane];
      cdt = pdt[p1 + lane];
      ctau = B - pc[p1 + lane];
    }
    if (l128 < (int)(p3 - p2)) {
      const int64_t p = p2 + l128;
      s_tri[slot][pidx[p] - g.j0] = make_int4(pdm[p], pdt[p], B - pc[p], 0);
    }
    const int nc = (int)(p2 - p1);
    const uint32_t* own = D + j * (int64_t)W;
#pragma unroll
    for (int k = 0; k < kDualK; k++) {
      const int x = l128 + kDualLanes * k;
      if (kDualLanes * k < cells) acc[k] = x < cells ? own[mb + x] : kNone;
    }
    // two cells of a thread and the block's eight pairs in flight together
#pragma unroll
    for (int k = 0; k < kDualK; k += 2) {
      if (kDualLanes * k >= cells) break;
      uint32_t v[2][kDualSlots];
#pragma unroll
      for (int q = 0; q < kDualSlots; q++) {
        const int32_t src = __builtin_amdgcn_readlane(csrc, q);
        const int32_t dm = __builtin_amdgcn_readlane(cdm, q);
        const int32_t tau = q < nc ? __builtin_amdgcn_readlane(ctau, q) : -1;
        const uint32_t* row = D + (int64_t)src * W;
#pragma unroll
        for (int h = 0; h < 2; h++) {
          const int x = l128 + kDualLanes * (k + h);
          const int32_t m = mb + x - dm;
          const bool ok = x < cells && m >= 0 && m <= tau;
          const uint32_t y = row[ok ? m : 0];
          v[h][q] = ok ? y : kNone;
        }
      }
#pragma unroll
      for (int q = 0; q < kDualSlots; q++) {
        const uint32_t dt = (uint32_t)__builtin_amdgcn_readlane(cdt, q);
#pragma unroll
        for (int h = 0; h < 2; h++)
          if (v[h][q] != kNone) acc[k + h] = dual_better<kTC>(acc[k + h], v[h][q] + dt);
      }
    }
  }
  for (int s = 0; s < nrows; s++) {
    if (slot == s) {                                      // the row is final
#pragma unroll
      for (int k = 0; k < kDualK; k++) {
        const int x = l128 + kDualLanes * k;
        if (x >= cells) continue;
        s_row[s][x] = acc[k];
        if (mb + x >= m0) D[j * (int64_t)W + mb + x] = acc[k];
      }
    }
    __syncthreads();
    if (slot <= s || slot >= nrows) continue;
    const int4 pr = s_tri[slot][s];
    if (pr.z < 0) continue;
#pragma unroll
    for (int k = 0; k < kDualK; k++) {
      const int x = l128 + kDualLanes * k;
      if (kDualLanes * k >= cells) break;
      const int y = x - pr.x;                             // left of the window: not needed
      const bool ok = x < cells && y >= 0 && mb + y <= pr.z;
      const uint32_t v = ok ? s_row[s][y] : kNone;
      if (v != kNone) acc[k] = dual_better<kTC>(acc[k], v + (uint32_t)pr.y);
    }
  }
}

// t of the objective over row V and the least m that attains it.
// host (pinned; null: none) receives the status.
__global__ __launch_bounds__(kDualThreads) void k_dual_select(const uint32_t* __restrict__ row,
                                                              int32_t W, int tc, DevStatus* st,
                                                              DevStatus* host) {
  __shared__ unsigned long long s_best;             // TC: t; MC: t + 1 (0: none)
  __shared__ int32_t s_m;
  if (threadIdx.x == 0) {
    s_best = tc ? (unsigned long long)kDualNone : 0ull;
    s_m = INT32_MAX;
  }
  __syncthreads();
  unsigned long long best = tc ? (unsigned long long)kDualNone : 0ull;
  for (int32_t m = threadIdx.x; m < W; m += blockDim.x) {
    const uint32_t x = row[m];
    if (tc ? x == kDualNone : x == 0u) continue;
    best = tc ? min(best, (unsigned long long)x) : max(best, (unsigned long long)x);
  }
  if (tc)
    atomicMin(&s_best, best);
  else
    atomicMax(&s_best, best);
  __syncthreads();
  const bool found = tc ? s_best != kDualNone : s_best != 0;
  if (found) {
    const uint32_t code = (uint32_t)s_best;
    for (int32_t m = threadIdx.x; m < W; m += blockDim.x)
      if (row[m] == code) {
        atomicMin(&s_m, m);
        break;
      }
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  DevStatus r = *st;
  r.t_sel = found ? (int32_t)(tc ? s_best : s_best - 1) : -1;
  r.m_sel = found ? s_m : -1;
  *st = r;
  if (host) *host = r;
}

// Traceback through the table (Section 4.2's, read on cells (L, m)): from
// (V, m*, t*), the next set is the smallest family index L among the pairs
// L < L' whose cell (L, m - dm) passes the budget test and holds t - dt (one
// always does along an optimal chain: its state there is reachable, and a
// better one would give a better optimum).  The walk must end at (empty set,
// 0, 0); then the chain's strategy is evaluated (finish_schedule).  The
// pairs of a step are scanned kDualTraceThreads at a time; the first hit in
// family order is the lowest hitting thread of the first chunk with one.
constexpr int kDualTraceThreads = 512;

template <bool kTC>
__global__ __launch_bounds__(kDualTraceThreads) void k_dual_trace(
    int64_t F, int n, int words, int64_t fstride, const uint64_t* __restrict__ bits,
    const uint64_t* __restrict__ bd, const int32_t* __restrict__ A, const int32_t* __restrict__ T,
    const int32_t* __restrict__ M, const int64_t* __restrict__ pred_ptr,
    const int32_t* __restrict__ pidx, const int32_t* __restrict__ pdt,
    const int32_t* __restrict__ pdm, const int32_t* __restrict__ pc, int32_t B, int32_t W,
    const uint32_t* __restrict__ D, int64_t T_total, DevStatus* st, int32_t* chain,
    ScheduleOut out) {
  constexpr int kWaves = kDualTraceThreads / 64;
  __shared__ int32_t s_first[2][kWaves];
  __shared__ int32_t s_src[2][kDualTraceThreads];
  __shared__ int32_t s_dt[2][kDualTraceThreads];
  __shared__ int32_t s_dm[2][kDualTraceThreads];
  __shared__ int32_t s_chain[kMaxNodes + 1];
  __shared__ int32_t s_M[kMaxNodes];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid / 64;
  // bring the pair lists, which every step reads, into this XCD's L2 first
  // when they are small (DenseNet-121's 267 steps: 321 -> 277 us)
  const int64_t P = pred_ptr[F];
  if (P <= ((int64_t)1 << 17)) {
    int32_t acc = 0;
    for (int64_t x = tid * 16; x < P; x += kDualTraceThreads * 16)
      acc ^= pidx[x] ^ pdt[x] ^ pc[x] ^ pdm[x];
    if (acc == 0x7fffffff) st->pad0 = acc;          // keeps the loads
  }
  int64_t j = F - 1;
  int64_t t = st->t_sel, m = st->m_sel;
  int32_t k = 0;
  bool bad = t < 0 || m < 0 || m >= W;
  int par = 0;
  while (j != 0 && !bad) {
    if (k >= F || k > n) {                          // each step removes a node
      bad = true;
      break;
    }
    const int64_t p0 = pred_ptr[j], p1 = pred_ptr[j + 1];
    int32_t next_i = -1, next_dt = 0, next_dm = 0;
    for (int64_t base = p0; base < p1 && next_i < 0; base += kDualTraceThreads) {
      const int64_t p = base + tid;
      const bool valid = p < p1;
      const int64_t pq = valid ? p : p0;
      const int32_t i = pidx[pq], dt = pdt[pq], dm = pdm[pq], c = pc[pq];
      const int64_t ms = m - dm;                     // memory before the step
      const bool ok = valid && ms >= 0 && ms <= B - c;
      const uint32_t x = D[(int64_t)i * W + (ok ? ms : 0)];
      const bool reached = kTC ? x != kDualNone : x != 0u;
      const int64_t tx = kTC ? (int64_t)x : (int64_t)x - 1;
      const bool hit = ok && reached && tx + dt == t;
      const unsigned long long bal = __ballot(hit);
      if (lane == 0) s_first[par][wave] = bal ? wave * 64 + __ffsll((long long)bal) - 1 : INT32_MAX;
      s_src[par][tid] = i;
      s_dt[par][tid] = dt;
      s_dm[par][tid] = dm;
      __syncthreads();
      int32_t f = INT32_MAX;
#pragma unroll
      for (int q = 0; q < kWaves; q++) f = min(f, s_first[par][q]);
      if (f != INT32_MAX) {
        next_i = s_src[par][f];
        next_dt = s_dt[par][f];
        next_dm = s_dm[par][f];
      }
      par ^= 1;
    }
    if (next_i < 0) {
      bad = true;
      break;
    }
    if (tid == 0) chain[k] = (int32_t)j;
    k++;
    t -= next_dt;
    m -= next_dm;
    j = next_i;
  }
  if (t != 0 || m != 0) bad = true;                  // the walk must end at (empty set, 0, 0)
  __syncthreads();
  finish_schedule<kDualTraceThreads>(bad ? -1 : k, n, words, fstride, bits, bd, A, T, M, T_total,
                                     chain, out, s_chain, s_M);
}

}  // namespace

// Rows per block of k_dual_block (8 or 4; 0: the halo leaves a workgroup's
// window, or blocks of 2 would fit, which cost more than levels) and every
// block's halo, the largest difference of M(L) over its sets.
int32_t dual_block_rows(int64_t F, const int32_t* Msum, std::vector<int32_t>* halo) {
  for (int32_t rows = kDualSlots; rows >= kDualSlots / 2; rows /= 2) {
    halo->clear();
    int32_t most = 0;
    for (int64_t j = 1; j < F; j += rows) {
      const auto mm = std::minmax_element(Msum + j, Msum + std::min<int64_t>(j + rows, F));
      halo->push_back(*mm.second - *mm.first);
      most = std::max(most, halo->back());
    }
    if (most <= kDualHalo) return rows;
  }
  halo->clear();
  return 0;
}

// Blocks where they take fewer microseconds of launches: a block about 10, a
// level about 3.6 (U-Net and the ladder keep their levels: 0.13 and 0.12 ms).
static bool dual_takes_blocks(rc_family f) {
  if (f->dual_rows == 0 || !f->dual_split) return false;
  const int64_t levels = (int64_t)f->level_ptr.size() - 2;
  const int64_t nblk = (f->F - 1 + f->dual_rows - 1) / f->dual_rows;
  return 10.0 * (double)nblk < 3.6 * (double)levels;
}

hipError_t launch_dual_trace(rc_family f, int32_t B, int32_t W, int objective, const uint32_t* D,
                             DevStatus* st, int32_t* chain, const ScheduleOut& out,
                             hipStream_t s) {
  rc_graph g = f->g;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(1), dim3(kDualTraceThreads), 0, s, f->F, g->n, g->words,
                       f->fstride, f->bits, f->bd, f->A, g->dT, g->dM, f->pred_ptr, f->pidx,
                       f->pdt, f->pdm, f->pc, B, W, D, g->T_total, st, chain, out);
  };
  if (objective == RC_TIME_CENTRIC)
    go(k_dual_trace<true>);
  else
    go(k_dual_trace<false>);
  return hipGetLastError();
}

hipError_t launch_dual(rc_family f, const std::vector<int64_t>& level_pairs, int32_t B, int32_t W,
                       int objective, uint32_t* D, DevStatus* st, DevStatus* host, hipEvent_t e0,
                       hipEvent_t e1, hipStream_t s) {
  const int64_t cells = f->F * (int64_t)W;
  const unsigned grid0 = (unsigned)std::min<int64_t>((cells + 255) / 256, 4096);
  const bool tc = objective == RC_TIME_CENTRIC;
  hipLaunchKernelGGL(k_dual_init, dim3(grid0), dim3(256), 0, s, D, cells, tc ? 1 : 0, st);
  if (e0 && hipEventRecord(e0, s) != hipSuccess) return hipErrorUnknown;
  const unsigned tiles = (unsigned)((W + kDualThreads - 1) / kDualThreads);
  const int64_t L = (int64_t)f->level_ptr.size() - 1;
  if (dual_takes_blocks(f)) {
    const int64_t R = f->dual_rows, nblk = (f->F - 1 + R - 1) / R;
    auto start = [&](int64_t b) { return std::min<int64_t>(1 + b * R, f->F); };
    for (int64_t b = 0; b < nblk; b++) {
      DualBlock g{};
      g.j0 = start(b);
      g.j1 = start(b + 1);
      g.n0 = g.j1;
      g.n1 = start(b + 2);
      g.halo = f->dual_halo[(size_t)b];
      g.row_blocks = (W + kDualOwn - 1) / kDualOwn;
      g.tiles = (int32_t)tiles;
      // a target's pairs from sources before block b: at most its position
      g.runs = (int32_t)((g.j0 + kDualRun - 1) / kDualRun);
      const int64_t items = (g.n1 - g.n0) * tiles * (int64_t)g.runs;   // below 2^31: F <= 8192
      const dim3 grid((unsigned)(g.row_blocks + (items + 3) / 4));
      if (tc)
        hipLaunchKernelGGL(k_dual_block<true>, grid, dim3(kDualSlots * kDualLanes), 0, s, g, W, B,
                           f->pred_ptr, f->dual_split, f->pidx, f->pdt, f->pdm, f->pc, D);
      else
        hipLaunchKernelGGL(k_dual_block<false>, grid, dim3(kDualSlots * kDualLanes), 0, s, g, W,
                           B, f->pred_ptr, f->dual_split, f->pidx, f->pdt, f->pdm, f->pc, D);
    }
  } else {
    for (int64_t l = 0; l < L; l++) {
      const int64_t lb = std::max<int64_t>(f->level_ptr[l], 1), le = f->level_ptr[l + 1];
      if (le <= lb) continue;
      const dim3 grid(tiles, (unsigned)(le - lb),
                      (unsigned)((level_pairs[l] + kDualPairs - 1) / kDualPairs));
      if (grid.z == 0) continue;
      if (tc)
        hipLaunchKernelGGL(k_dual_level<true>, grid, dim3(kDualThreads), 0, s, lb, W, B,
                           f->pred_ptr, f->pidx, f->pdt, f->pdm, f->pc, D);
      else
        hipLaunchKernelGGL(k_dual_level<false>, grid, dim3(kDualThreads), 0, s, lb, W, B,
                           f->pred_ptr, f->pidx, f->pdt, f->pdm, f->pc, D);
    }
  }
  if (e1 && hipEventRecord(e1, s) != hipSuccess) return hipErrorUnknown;
  hipLaunchKernelGGL(k_dual_select, dim3(1), dim3(kDualThreads), 0, s,
                     D + (f->F - 1) * (int64_t)W, W, tc ? 1 : 0, st, host);
  return hipGetLastError();
}

}  // namespace rcdp
