// The DP of Section 4.2 / Appendix A (Algorithm 1) on the device: table
// fill, selection of t*, traceback of optarg and re-evaluation of the
// resulting canonical strategy with Eq. 1 and Eq. 2.
//
// Table layout: one row per family member L, holding the cells
// t = 0 .. w_L - 1 (w_L = T(L \ boundary(L)) + 1; every cell beyond is
// provably infinite, since each recomputed node of a chain ending at L lies
// in L \ boundary(L)).  Rows are contiguous in t and end on 128-byte
// lines.  A cell stores m = opt[L, t] as uint16 (0xFFFF = infinity), or
// as uint32 (0xFFFFFFFF = infinity) for budgets beyond the 16-bit range
// (the level fill, selection, traceback and export take either width).
//
// Pull form of Algorithm 1: opt[L', t'] is the minimum over predecessors
// L (proper subsets of L' in the family) of opt[L, t' - dt] + dm, taken
// over the sources that pass the budget test opt[L, t] + c <= B.
//
// optarg is not stored by the fill.  Algorithm 1's strict update over
// ascending sources makes optarg[L', t'] the smallest family index L among
// the predecessors whose cell passes the budget test and reproduces
// opt[L', t'] (the first source to reach the minimum writes it, later ones
// only tie).  That rule is evaluated where optarg is needed: at every step
// of the traceback (k_trace) and, for a whole-table export, by k_arg_all.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "rc_internal.h"
#include "schedule.h"
#include "wavefront.h"

namespace rcdp {

namespace {

constexpr int kWave = 64;
constexpr int kFillThreads = 256;
constexpr int kCellsPerThread = 4;
constexpr int kTile = kFillThreads * kCellsPerThread;

// Infinity of a table of cells of type T.
template <class T>
__device__ __forceinline__ constexpr uint32_t cell_inf() {
  return sizeof(T) == 2 ? 0xFFFFu : 0xFFFFFFFFu;
}

// Tables of one launch (z, or y of the selection).
constexpr int kTables = 64;
struct InitTables {
  void* m[kTables];
  DevStatus* st[kTables];
  uint16_t* sentinel[kTables];
};
struct SelectTables {
  const void* m[kTables];
  DevStatus* st[kTables];
  DevStatus* host;
};

// opt[empty, 0] = 0 (Algorithm 1's initial condition), the selection state,
// infinity in the padding (the cells of every row's slot before the row, at
// least kGuard, the kGuard cells after the last row and an 8-cell sentinel,
// so that a window that overlaps a row reads infinity outside it) and, with
// pend, kPendM ("not written yet") in every cell after row 0.  Block (x, y):
// kInitChunk cells of row lb + y's slot, 16 bytes per store.
constexpr int kInitChunk = 16384;

template <class T>
__global__ __launch_bounds__(kFillThreads) void k_solve_init(InitTables tabs, int64_t lb,
                                                             int64_t F,
                                                             const int32_t* __restrict__ w,
                                                             const int64_t* __restrict__ row_off,
                                                             int64_t cells, int objective,
                                                             int pend) {
  constexpr int kVec = 16 / (int)sizeof(T);
  T* const m = static_cast<T*>(tabs.m[blockIdx.z]);
  const int64_t s = lb + blockIdx.y;
  const int32_t ws = w[s];
  const int64_t off = row_off[s];
  const int64_t slot = row_slot(ws);
  const int64_t pad = slot - ws;                    // padding cells of the slot
  const int64_t end = pend && s > 0 ? slot : pad;   // cells of the slot to write
  T* const p = m + off - pad;                       // 128-byte aligned
  for (int64_t x = (int64_t)blockIdx.x * kInitChunk + kVec * threadIdx.x;
       x < min(end, ((int64_t)blockIdx.x + 1) * kInitChunk); x += kVec * kFillThreads) {
    union {
      uint4 q;
      T c[kVec];
    } v;
#pragma unroll
    for (int k = 0; k < kVec; k++) v.c[k] = x + k < pad ? (T)cell_inf<T>() : (T)kPendM;
    if (x + kVec <= end) {
      *reinterpret_cast<uint4*>(p + x) = v.q;
    } else {
#pragma unroll
      for (int k = 0; k < kVec; k++)
        if (x + k < end) p[x + k] = v.c[k];
    }
  }
  if (blockIdx.x != 0) return;
  if (s == F - 1)
    for (int64_t x = cells + threadIdx.x; x < cells + kGuard; x += kFillThreads)
      m[x] = (T)cell_inf<T>();
  if (s != 0) return;
  if (threadIdx.x < 8 && tabs.sentinel[blockIdx.z])
    tabs.sentinel[blockIdx.z][threadIdx.x] = (uint16_t)kInfM;
  if (threadIdx.x == 0) {
    DevStatus* const st = tabs.st[blockIdx.z];
    m[off] = 0;
    st->error = 0;
    st->t_sel = objective == RC_TIME_CENTRIC ? INT32_MAX : -1;
    st->m_sel = -1;
    st->k = 0;
    st->done = 0;
  }
}

// One launch per size level (targets of equal size never contain each
// other).  Block (x, y): cells [x * kTile, (x + 1) * kTile) of target
// lb + y; each thread owns kCellsPerThread cells strided by the block size
// so that every source read and every store of a wave is contiguous.
template <class T>
__global__ __launch_bounds__(kFillThreads) void k_fill_level(
    int64_t lb, const int32_t* __restrict__ w, const int64_t* __restrict__ row_off,
    const int64_t* __restrict__ pred_ptr, const int32_t* __restrict__ pidx,
    const int32_t* __restrict__ pdt, const int32_t* __restrict__ pdm,
    const int32_t* __restrict__ pc, int32_t Beff, T* __restrict__ m) {
  const int64_t j = lb + blockIdx.y;
  const int32_t wj = w[j];
  const int32_t tile0 = blockIdx.x * kTile;
  if (tile0 >= wj) return;
  uint32_t acc[kCellsPerThread];
#pragma unroll
  for (int r = 0; r < kCellsPerThread; r++) acc[r] = cell_inf<T>();
  const int64_t p0 = pred_ptr[j], p1 = pred_ptr[j + 1];
  for (int64_t p = p0; p < p1; ++p) {
    // budget test of Algorithm 1: opt[L, t] + c <= B, i.e. opt[L, t] <= tau
    const int32_t tau = Beff - pc[p];
    if (tau < 0) continue;                    // no source cell can pass
    const int32_t dt = pdt[p];
    const int32_t i = pidx[p];
    const int32_t wi = w[i];                  // cells of the source row
    // window misses the tile (whose end may lie past the last int32)
    if (dt >= (int64_t)tile0 + kTile || dt + wi <= tile0) continue;
    const T* src = m + row_off[i];
    const uint32_t dm = (uint32_t)pdm[p];
#pragma unroll
    for (int r = 0; r < kCellsPerThread; r++) {
      const int32_t t = tile0 + r * kFillThreads + (int32_t)threadIdx.x - dt;
      if ((uint32_t)t < (uint32_t)wi) {
        const uint32_t x = src[t];
        if (x <= (uint32_t)tau) acc[r] = min(acc[r], x + dm);
      }
    }
  }
  T* mo = m + row_off[j];
#pragma unroll
  for (int r = 0; r < kCellsPerThread; r++) {
    const int32_t tp = tile0 + r * kFillThreads + (int32_t)threadIdx.x;
    if (tp < wj) mo[tp] = (T)acc[r];
  }
}

// The level fill, 16 bytes of cells per lane (eight 16-bit cells, two per
// packed instruction, or four 32-bit cells).  Cells are counted from the
// row's end, which lies on a kRowAlign boundary: lane g of target j owns the
// kVec cells from t = w_j - kVec (g + 1) on, one aligned 16-byte store.
// Along a pair its source cells are the kVec cells from t - dt on, one
// 16-byte load at whatever alignment that has (aligned loads of two words
// and a shift cost three times the instructions); t - dt is clamped to
// [-kVec, w_i], where the load reads the source row's padding, infinity, so
// no cell is masked.
//
// The NW waves of a workgroup own the same cells and split the pairs: lane l
// of wave v holds the record of pair 64 NW r + NW l + v of round r (the next
// round's in flight), the wave votes which of its 64 pairs pass the budget
// at all and overlap the tile, and takes those kLevelGroup at a time: the
// record's words to scalar registers, every load of the group out before
// the first is used, then the relaxations.  The waves' minima meet in LDS.
// Bound by each wave's chain of groups (one load latency each) on small
// levels and by the source reads on long rows; measured at launch_level_vec.
constexpr int kLevelGroup = 8;
static_assert(sizeof(LevelPair) == 32, "a record is two 16-byte loads");

template <class T>
struct LevelCells;
template <>
struct LevelCells<uint16_t> {
  uint32_t v[4];
  // r = min(acc, x + dm where x <= tau), all as packed pairs
  __device__ __forceinline__ void relax(const LevelCells& x, uint32_t tau, uint32_t dm) {
    using wf::u16x2;
    const u16x2 tv = __builtin_bit_cast(u16x2, tau * 0x10001u);
    const u16x2 dv = __builtin_bit_cast(u16x2, dm * 0x10001u);
#pragma unroll
    for (int k = 0; k < 4; k++)
      v[k] = __builtin_bit_cast(uint32_t, wf::relax2(__builtin_bit_cast(u16x2, v[k]),
                                                     __builtin_bit_cast(u16x2, x.v[k]), tv, dv));
  }
  __device__ __forceinline__ void merge(const LevelCells& x) {
    using wf::u16x2;
#pragma unroll
    for (int k = 0; k < 4; k++)
      v[k] = __builtin_bit_cast(
          uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, v[k]),
                                              __builtin_bit_cast(u16x2, x.v[k])));
  }
};
template <>
struct LevelCells<uint32_t> {
  uint32_t v[4];
  __device__ __forceinline__ void relax(const LevelCells& x, uint32_t tau, uint32_t dm) {
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = min(v[k], x.v[k] <= tau ? x.v[k] + dm : 0xFFFFFFFFu);
  }
  __device__ __forceinline__ void merge(const LevelCells& x) {
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = min(v[k], x.v[k]);
  }
};

// 16 bytes at any alignment of a cell.
typedef uint32_t u32x4_at2 __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x4_at4 __attribute__((ext_vector_type(4), aligned(4)));

template <class T>
__device__ __forceinline__ LevelCells<T> load_cells(const char* base, int32_t off) {
  typedef typename std::conditional<sizeof(T) == 2, u32x4_at2, u32x4_at4>::type V;
  const V q = *reinterpret_cast<const V*>(base + (uint32_t)off);
  LevelCells<T> r;
  r.v[0] = q.x;
  r.v[1] = q.y;
  r.v[2] = q.z;
  r.v[3] = q.w;
  return r;
}

// Tile `tile` of target j, over its pairs [p0, p1); the whole workgroup calls
// it.  s_acc: NW - 1 waves of LDS.
template <class T, int NW>
__device__ __forceinline__ void level_tile(int32_t tile, int32_t wj, int64_t rj,
                                           int64_t p0, int64_t p1,
                                           const LevelPair* __restrict__ lp, int32_t Beff,
                                           T* m, LevelCells<T> (*s_acc)[kWave]) {
  constexpr int kB = (int)sizeof(T);
  constexpr int kVec = 16 / kB;
  constexpr int kTileCells = kWave * kVec;
  const int32_t hi_t = wj - tile * kTileCells;         // the tile is [hi_t - kTileCells, hi_t)
  if (hi_t <= 0) return;                               // the whole workgroup leaves
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const int32_t t0 = hi_t - kVec * (lane + 1);                   // the lane's first cell
  LevelCells<T> acc = {{~0u, ~0u, ~0u, ~0u}};
  typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
  typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
  auto record = [&](int64_t p, i32x4& a, i32x2& b) {
    const LevelPair* r = lp + (p < p1 ? p : p0);
    a = *reinterpret_cast<const i32x4*>(r);
    b = *reinterpret_cast<const i32x2*>(&r->c);
  };
  int64_t p = p0 + (int64_t)lane * NW + wave;
  i32x4 na;                                                      // the next round's record
  i32x2 nb;
  if (p0 < p1) record(p, na, nb);
  for (int64_t r0 = p0; r0 < p1; r0 += NW * kWave, p += NW * kWave) {
    const i32x4 a = na;                         // lo (64 bits), dt, w
    const i32x2 b = nb;                         // c, dm
    const bool valid = p < p1;
    if (r0 + NW * kWave < p1) record(p + NW * kWave, na, nb);
    // the pair's window overlaps the tile and some source cell can pass
    unsigned long long live = __ballot(valid && Beff >= b.x && a.z < hi_t &&
                                       a.z + a.w > hi_t - kTileCells);
    // G pairs at a time; past the last live pair that pair again, which
    // changes nothing and keeps every load and relaxation unconditional
    auto group = [&](auto G) __attribute__((always_inline)) {
      constexpr int kG = decltype(G)::value;
      LevelCells<T> x[kG];
      uint32_t tau[kG], dm[kG];
      int k = 0;
#pragma unroll
      for (int q = 0; q < kG; q++) {
        if (live) k = __builtin_ctzll(live);
        live &= live - 1;
        const uint64_t lo = (uint32_t)__builtin_amdgcn_readlane(a.x, k) |
                            ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(a.y, k) << 32);
        const int32_t dt = __builtin_amdgcn_readlane(a.z, k);
        const int32_t ws = __builtin_amdgcn_readlane(a.w, k);
        tau[q] = (uint32_t)(Beff - __builtin_amdgcn_readlane(b.x, k));
        dm[q] = (uint32_t)__builtin_amdgcn_readlane(b.y, k);
        // offsets from kVec cells before the row, never negative
        const char* base = reinterpret_cast<const char*>(m) + ((int64_t)lo - kVec) * kB;
        x[q] = load_cells<T>(base, (min(max(t0 - dt, -kVec), ws) + kVec) * kB);
      }
#pragma unroll
      for (int q = 0; q < kG; q++) acc.relax(x[q], tau[q], dm[q]);
    };
    while (live) {
      const int cnt = __popcll(live);
      if (cnt > kLevelGroup / 2)
        group(std::integral_constant<int, kLevelGroup>{});
      else if (cnt > kLevelGroup / 4)
        group(std::integral_constant<int, kLevelGroup / 2>{});
      else
        group(std::integral_constant<int, kLevelGroup / 4>{});
    }
  }
  if (wave > 0) s_acc[wave - 1][lane] = acc;
  if (NW > 1) __syncthreads();
  if (wave > 0 || t0 + kVec <= 0) return;
#pragma unroll
  for (int q = 0; q < NW - 1; q++) acc.merge(s_acc[q][lane]);
  union {
    uint4 q;
    T c[kVec];
  } o;
  o.q = make_uint4(acc.v[0], acc.v[1], acc.v[2], acc.v[3]);
  if (t0 < 0) {                                      // cells before t = 0: padding, infinite
#pragma unroll
    for (int c = 0; c < kVec; c++)
      if (t0 + c < 0) o.c[c] = (T)cell_inf<T>();
  }
  *reinterpret_cast<uint4*>(m + rj + t0) = o.q;
}

template <class T, int NW>
__global__ __launch_bounds__(NW * kWave) void k_fill_level_vec(
    int64_t lb, const int32_t* __restrict__ w, const int64_t* __restrict__ row_off,
    const int64_t* __restrict__ pred_ptr, const LevelPair* __restrict__ lp, int32_t Beff,
    T* __restrict__ m) {
  __shared__ LevelCells<T> s_acc[NW > 1 ? NW - 1 : 1][kWave];
  const int64_t j = lb + blockIdx.y;
  level_tile<T, NW>((int32_t)blockIdx.x, w[j], row_off[j], pred_ptr[j], pred_ptr[j + 1], lp, Beff,
                    m, s_acc);
}

// The block fill, for narrow tables of many levels: one launch per kFbRows
// consecutive targets.  Rows are right-aligned, x = the distance of a cell
// from its row's end; along a pair the target cell x reads the source cell
// x - e, e = P_j - P_i - dt >= 0 (P = w - 1).  Launch b has two kinds of
// workgroups, beside each other:
//  - panel (block b + 1): the pairs from sources before block b, final by now,
//    as a tile of the level fill; the minima lie in the table itself;
//  - rows (block b): for kFbOwn cells, the rows start from their panel (the
//    launch before), take the pairs from the previous block's rows, then
//    finish one after the other in LDS, each relaxing the later rows.
// A step reads cells closer to the row's end only, so a rows workgroup
// recomputes the `halo` cells to the right of its own instead of waiting for
// their owner: along a path inside the block the shifts sum to at most
// P_last - P_first (every dt >= 0), and the host passes the largest
// difference of P over the block.  Halo cells are stored final by their owner
// meanwhile; reading either value gives the same minimum.
//
// A slot of one wave per target, a lane up to kFbK cells, in registers; one
// barrier per row.  Bound by a launch's chain of cold loads and by the
// instructions of the sixteen waves of a rows workgroup, so few own cells and
// many workgroups are best although they repeat more of the halo:
// densenet121_t10 (27 blocks, halos of 31 to 271 cells) 0.29 ms with 32 own
// cells, 0.32 with 64, 0.42 with 128, 0.54 with 256; the split-panel
// wavefront, 2 us a row whatever the row's length, 0.92.
constexpr int kFbRows = 16;
constexpr int kFbOwn = 32;
constexpr int kFbK = 14;
constexpr int kFbSpan = kFbK * kWave;
constexpr int kFbHalo = kFbSpan - kFbOwn;
constexpr int kFbThreads = kFbRows * kWave;

struct FbTables {
  uint16_t* m[kTables];
  int32_t Beff[kTables];
};
struct FbBlock {
  int64_t j0, j1;             // rows of the block
  int64_t n0, n1;             // rows of the next block
  int32_t halo, row_blocks;   // rows workgroups
  int32_t tiles;              // panel: tiles of a target
};

__global__ __launch_bounds__(kFbThreads) void k_fill_block(
    FbTables tabs, FbBlock g, const int32_t* __restrict__ w, const int64_t* __restrict__ row_off,
    const int64_t* __restrict__ pred_ptr, const int64_t* __restrict__ split,
    const int32_t* __restrict__ pidx, const int32_t* __restrict__ pdt,
    const int32_t* __restrict__ pdm, const int32_t* __restrict__ pc,
    const LevelPair* __restrict__ lp) {
  __shared__ LevelCells<uint16_t> s_acc[kFbRows - 1][kWave];
  __shared__ uint16_t s_row[kFbRows][kFbSpan];
  __shared__ int4 s_tri[kFbRows][kFbRows];      // [target][source] e, dm, B - c (-1: none)
  uint16_t* const m = tabs.m[blockIdx.y];
  const int32_t Beff = tabs.Beff[blockIdx.y];
  const int tid = threadIdx.x;
  if ((int32_t)blockIdx.x >= g.row_blocks) {
    const int32_t item = (int32_t)blockIdx.x - g.row_blocks;
    const int64_t j = g.n0 + item / g.tiles;
    level_tile<uint16_t, kFbRows>(item % g.tiles, w[j], row_off[j], pred_ptr[j], split[2 * j], lp,
                                  Beff, m, s_acc);
    return;
  }
  const int slot = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid & (kWave - 1);
  const int nrows = (int)(g.j1 - g.j0);
  const int64_t j = g.j0 + slot;
  const int32_t x0 = (int32_t)blockIdx.x * kFbOwn;
  const int32_t xb = max(0, x0 - g.halo);                 // first cell computed
  const int32_t cells = x0 + kFbOwn - xb;                 // at most kFbSpan
  if (tid < kFbRows * kFbRows) s_tri[tid / kFbRows][tid % kFbRows].z = -1;
  uint32_t acc[kFbK];
#pragma unroll
  for (int k = 0; k < kFbK; k++) acc[k] = kInfM;
  __syncthreads();
  int32_t wj = 0;
  int64_t end = 0;
  if (slot < nrows) {
    wj = w[j];
    end = row_off[j] + wj - 1;
    const int64_t p1 = split[2 * j], p2 = split[2 * j + 1], p3 = pred_ptr[j + 1];
    // lane q: the q-th pair from the previous block's rows, and from the block's
    int32_t cend = 0, ce = 0, cp = 0, cdm = 0, ctau = -1;
    if (lane < (int)(p2 - p1)) {
      const int32_t i = pidx[p1 + lane];
      const int32_t wi = w[i];
      cend = (int32_t)(row_off[i] + wi - 1);
      ce = wj - wi - pdt[p1 + lane];
      cp = wi;
      cdm = pdm[p1 + lane];
      ctau = Beff - pc[p1 + lane];
    }
    if (lane < (int)(p3 - p2)) {
      const int64_t p = p2 + lane;
      const int32_t i = pidx[p];
      s_tri[slot][i - g.j0] = make_int4(wj - w[i] - pdt[p], pdm[p], Beff - pc[p], 0);
    }
    if (g.j0 > 1) {                                       // block 0 has no panel
#pragma unroll
      for (int k = 0; k < kFbK; k++) {
        const int x = xb + lane + kWave * k;
        if (kWave * k < cells) acc[k] = m[end - min(x, wj)];   // x = wj: padding, infinite
      }
    }
    // the pairs from the previous block for H cells of a lane, their sixteen
    // loads each in flight together; a source cell outside its row is read in
    // its padding
    const int nc = (int)(p2 - p1);
    auto cross = [&](auto H, uint32_t* a, int32_t x) __attribute__((always_inline)) {
      constexpr int kH = decltype(H)::value;
      uint32_t v[kH][kFbRows];
#pragma unroll
      for (int q = 0; q < kFbRows; q++) {
        const int32_t e = __builtin_amdgcn_readlane(ce, q);
        const int32_t pe = __builtin_amdgcn_readlane(cp, q);
        const int32_t qe = __builtin_amdgcn_readlane(cend, q);
#pragma unroll
        for (int h = 0; h < kH; h++) v[h][q] = m[qe - min(max(x + kWave * h - e, -1), pe)];
      }
#pragma unroll
      for (int q = 0; q < kFbRows; q++) {
        const int32_t tau = __builtin_amdgcn_readlane(ctau, q);     // -1 past the list
        const uint32_t dm = (uint32_t)__builtin_amdgcn_readlane(cdm, q);
#pragma unroll
        for (int h = 0; h < kH; h++)
          a[h] = min(a[h], (int32_t)v[h][q] <= tau ? v[h][q] + dm : kInfM);
      }
    };
    if (nc > 0) {
      if (cells <= kWave) {
        cross(std::integral_constant<int, 1>{}, &acc[0], xb + lane);
      } else {
#pragma unroll
        for (int k = 0; k < kFbK; k += 2) {
          if (kWave * k >= cells) break;
          cross(std::integral_constant<int, 2>{}, &acc[k], xb + lane + kWave * k);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kFbK; k++)
      if (xb + lane + kWave * k >= wj) acc[k] = kInfM;
  }
  for (int s = 0; s < nrows; s++) {
    if (slot == s) {                                      // the row is final
#pragma unroll
      for (int k = 0; k < kFbK; k++) {
        if (kWave * k >= cells) break;
        const int y = lane + kWave * k;
        s_row[s][y] = (uint16_t)acc[k];
        const int x = xb + y;
        if (x >= x0 && y < cells && x < wj) m[end - x] = (uint16_t)acc[k];
      }
    }
    __syncthreads();
    if (slot <= s || slot >= nrows) continue;
    const int4 pr = s_tri[slot][s];
    if (pr.z < 0) continue;
#pragma unroll
    for (int k = 0; k < kFbK; k++) {
      if (kWave * k >= cells) break;
      const int y = lane + kWave * k - pr.x;              // left of the window: not needed
      const uint32_t v = y >= 0 ? s_row[s][y] : kInfM;
      if ((int32_t)v <= pr.z && xb + lane + kWave * k < wj)
        acc[k] = min(acc[k], v + (uint32_t)pr.y);
    }
  }
}

// The level fill's record of each pair (built once per family).
__global__ void k_level_pairs(int64_t P, const int32_t* __restrict__ pidx,
                              const int32_t* __restrict__ pdt, const int32_t* __restrict__ pdm,
                              const int32_t* __restrict__ pc, const int32_t* __restrict__ w,
                              const int64_t* __restrict__ row_off, LevelPair* lp) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= P) return;
  const int32_t i = pidx[p];
  lp[p] = LevelPair{row_off[i], pdt[p], w[i], pc[p], pdm[p], 0, 0};
}

// The dominance skip of Section 4.2 (last paragraph): a cell t of row L is
// never propagated when an earlier cell of the same row holds strictly less
// memory.  Such a cell is stored as infinity, which leaves each row as its
// weak front (the cells with m no larger than every earlier m), the only
// cells that the selection of t* or the traceback reads.
//
// The fronts are taken from the whole finished table, not level by level: a
// front cell's value comes from a front cell (a dominated source cell has an
// earlier cell with strictly less memory, which passes the same budget test
// and lands earlier on the target with strictly less), so a row's front is
// the same whether the rows before it were reduced or not, and the table is
// filled by the fastest path with no order between a row's front and the
// rows after it.
//
// Two passes over segments of kSeg cells, a workgroup each (rows lb + y):
// k_front_min stores each segment's least m; k_front takes the least m of
// the row's segments before its own as the carry and scans its own.  A
// thread owns 8 consecutive cells, one 16-byte load and at most one such
// store.  Bound by the table's bytes, read twice: U-Net's 61 M cells 28 and
// 49 us (4.4 TB/s of reads in the first); two launches after every size
// level, with the carry read by every thread, took 225 us and 1.72 ms.
// Segment x of row j, counted from the row's first cell
// rounded down to 8 cells, has the slot (row_off[j] >> kSegShift) + j + x.
constexpr int kSegShift = 11;
constexpr int kSeg = 1 << kSegShift;
static_assert(kSeg == 8 * kFillThreads, "eight cells per thread");

// The cells of segment blockIdx.x of row j that a thread owns, outside the
// row infinite; t = the first one's t.
__device__ __forceinline__ uint16_t* front_cells(int64_t off, int32_t wj, uint16_t* m, int32_t& t,
                                                 uint16_t (&c)[8]) {
  const int32_t a = (int32_t)(off & 7);
  t = (int32_t)blockIdx.x * kSeg + 8 * (int32_t)threadIdx.x - a;
  uint16_t* p = m + off + t;
  union {
    uint4 q;
    uint16_t v[8];
  } x;
  x.q = make_uint4(~0u, ~0u, ~0u, ~0u);
  if (t < wj) x.q = *reinterpret_cast<const uint4*>(p);
#pragma unroll
  for (int k = 0; k < 8; k++) c[k] = t + k >= 0 && t + k < wj ? x.v[k] : (uint16_t)kInfM;
  return p;
}

__global__ __launch_bounds__(kFillThreads) void k_front_min(
    int64_t lb, const int32_t* __restrict__ w, const int64_t* __restrict__ row_off,
    uint16_t* __restrict__ m, uint16_t* __restrict__ segmin) {
  __shared__ uint32_t s_wave[kFillThreads / kWave];
  const int64_t j = lb + blockIdx.y;
  const int32_t wj = w[j];
  const int64_t off = row_off[j];
  if ((int64_t)blockIdx.x * kSeg >= wj + (off & 7)) return;   // the whole block leaves together
  int32_t t;
  uint16_t c[8];
  front_cells(off, wj, m, t, c);
  uint32_t x = kInfM;
#pragma unroll
  for (int k = 0; k < 8; k++) x = min(x, (uint32_t)c[k]);
  for (int o = kWave / 2; o > 0; o >>= 1) x = min(x, (uint32_t)__shfl_xor(x, o, kWave));
  if (threadIdx.x % kWave == 0) s_wave[threadIdx.x / kWave] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < kFillThreads / kWave; q++) x = min(x, s_wave[q]);
    segmin[(off >> kSegShift) + j + blockIdx.x] = (uint16_t)x;
  }
}

__global__ __launch_bounds__(kFillThreads) void k_front(
    int64_t lb, const int32_t* __restrict__ w, const int64_t* __restrict__ row_off,
    uint16_t* __restrict__ m, const uint16_t* __restrict__ segmin) {
  __shared__ uint32_t s_carry[kFillThreads / kWave], s_wave[kFillThreads / kWave];
  const int64_t j = lb + blockIdx.y;
  const int32_t wj = w[j];
  const int64_t off = row_off[j];
  if ((int64_t)blockIdx.x * kSeg >= wj + (off & 7)) return;   // the whole block leaves together
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  int32_t t;
  uint16_t c[8];
  uint16_t* p = front_cells(off, wj, m, t, c);
  // least m of the segments before, over the workgroup
  uint32_t before = kInfM;
  const uint16_t* sm = segmin + (off >> kSegShift) + j;
  for (uint32_t q = threadIdx.x; q < blockIdx.x; q += kFillThreads)
    before = min(before, (uint32_t)sm[q]);
  for (int o = kWave / 2; o > 0; o >>= 1)
    before = min(before, (uint32_t)__shfl_xor(before, o, kWave));
  uint32_t own = kInfM;                     // least of the thread's cells, then of the lanes before
#pragma unroll
  for (int k = 0; k < 8; k++) own = min(own, (uint32_t)c[k]);
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t y = __shfl_up(own, o, kWave);
    if (lane >= o) own = min(own, y);
  }
  if (lane == kWave - 1) {
    s_carry[wave] = before;
    s_wave[wave] = own;
  }
  uint32_t least = __shfl_up(own, 1, kWave);
  if (lane == 0) least = kInfM;
  __syncthreads();
  for (int q = 0; q < kFillThreads / kWave; q++) {
    least = min(least, s_carry[q]);
    if (q < wave) least = min(least, s_wave[q]);
  }
  // one 16-byte store; the cells before the row's first one are padding
  union {
    uint4 q;
    uint16_t v[8];
  } x;
  bool changed = false;
#pragma unroll
  for (int k = 0; k < 8; k++) {
    const bool dominated = c[k] > least;
    x.v[k] = dominated ? (uint16_t)kInfM : c[k];
    changed |= dominated && c[k] != kInfM;
    least = min(least, (uint32_t)c[k]);
  }
  if (changed) *reinterpret_cast<uint4*>(p) = x.q;
}

// optarg of every cell from the final table: the smallest predecessor index
// whose cell passes the budget test and reproduces the target value
// (Algorithm 1's first writer).
template <class T>
__global__ __launch_bounds__(kFillThreads) void k_arg_all(
    int64_t lb, const int32_t* __restrict__ w, const int64_t* __restrict__ row_off,
    const int64_t* __restrict__ pred_ptr, const int32_t* __restrict__ pidx,
    const int32_t* __restrict__ pdt, const int32_t* __restrict__ pdm,
    const int32_t* __restrict__ pc, int32_t Beff, const T* __restrict__ m,
    uint16_t* __restrict__ arg) {
  const int64_t j = lb + blockIdx.y;
  const int32_t wj = w[j];
  const int32_t tp = blockIdx.x * kFillThreads + threadIdx.x;
  if (tp >= wj) return;
  const uint32_t mj = m[row_off[j] + tp];
  uint32_t a = kNoArg;
  if (mj != cell_inf<T>() && j > 0) {
    for (int64_t p = pred_ptr[j]; p < pred_ptr[j + 1]; ++p) {
      const int32_t t = tp - pdt[p];
      const int32_t i = pidx[p];
      if ((uint32_t)t >= (uint32_t)w[i]) continue;
      const uint32_t x = m[row_off[i] + t];
      if (x != cell_inf<T>() && (int64_t)x <= (int64_t)Beff - pc[p] &&
          (uint32_t)(x + pdm[p]) == mj) {
        a = (uint32_t)i;
        break;
      }
    }
  }
  arg[row_off[j] + tp] = (uint16_t)a;
}

// t* = min (time-centric) or max (memory-centric) finite t of row V, and
// opt[V, t*].  A lane reads 16 bytes of the row at a time, counted from the
// row's end (aligned to kRowAlign cells); a workgroup reduces to one atomic,
// and the last workgroup to finish (st->done) reads the result back and
// writes the status to the host's pinned buffer.  Table y of tabs.  Bound
// by its loads in flight: U-Net's 2.4 M cells take 10 us (13 with 512
// workgroups, whose atomics meet on one address), against 48 us with one
// cell per load and 64 workgroups and 5 more in a second launch.
constexpr int kSelectThreads = 256;
constexpr int kSelectBlocks = 128;

template <class T>
__global__ __launch_bounds__(kSelectThreads) void k_select(SelectTables tabs,
                                                          const int64_t* row_off, int64_t v,
                                                          const int32_t* w, int objective) {
  constexpr int kVec = 16 / (int)sizeof(T);
  const T* const m = static_cast<const T*>(tabs.m[blockIdx.y]);
  DevStatus* const st = tabs.st[blockIdx.y];
  __shared__ int32_t s_best[kSelectThreads / kWave];
  const int64_t off = row_off[v];
  const int32_t wv = w[v];
  const bool tc = objective == RC_TIME_CENTRIC;
  int32_t best = tc ? INT32_MAX : -1;
  // a row has up to 2^31 - 2 cells: its rounded length is no int32
  const int32_t groups = (int32_t)(((int64_t)wv + kVec - 1) / kVec);
  for (int32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < groups;
       g += gridDim.x * blockDim.x) {
    const int32_t t0 = (int32_t)(wv - kVec * ((int64_t)g + 1));   // before the row for the last g
    union {
      uint4 q;
      T c[kVec];
    } x;
    x.q = *reinterpret_cast<const uint4*>(m + off + t0);
#pragma unroll
    for (int k = 0; k < kVec; k++)
      if (t0 + k >= 0 && x.c[k] != (T)cell_inf<T>())
        best = tc ? min(best, t0 + k) : max(best, t0 + k);
  }
  for (int o = kWave / 2; o > 0; o >>= 1) {
    const int32_t y = __shfl_xor(best, o, kWave);
    best = tc ? min(best, y) : max(best, y);
  }
  if ((threadIdx.x & (kWave - 1)) == 0) s_best[threadIdx.x / kWave] = best;
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int q = 1; q < kSelectThreads / kWave; q++)
    best = tc ? min(best, s_best[q]) : max(best, s_best[q]);
  if (tc ? best != INT32_MAX : best >= 0) {
    if (tc)
      atomicMin(&st->t_sel, best);
    else
      atomicMax(&st->t_sel, best);
  }
  __threadfence();
  if (atomicAdd(&st->done, 1) != (int32_t)gridDim.x - 1) return;
  __threadfence();
  int32_t t = __hip_atomic_load(&st->t_sel, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (t == INT32_MAX) t = -1;
  DevStatus r = *st;
  r.t_sel = t;
  r.m_sel = t >= 0 ? (int32_t)m[off + t] : -1;
  st->t_sel = r.t_sel;
  st->m_sel = r.m_sel;
  tabs.host[blockIdx.y] = r;
}

// Traceback from (V, t*) (Section 4.2), then Eq. 1 and Eq. 2 of the chain
// from their definitions: U_i is the union of boundaries of L_1..L_i,
// segment i needs M(U_{i-1}) + 2 M(V_i) + A(L_i), the overhead is
// T(V \ U_k).  At each step the workgroup scans the predecessors of L'
// (ascending family index, kTraceThreads at a time) for optarg[L', t']:
// the smallest index whose cell passes the budget test and reproduces the
// target value.
constexpr int kTraceThreads = 512;
constexpr int kTraceLds = 2048;       // families up to this size keep their per-set arrays in LDS

template <bool kLds, class Cell>
__global__ __launch_bounds__(kTraceThreads) void k_trace(
    int64_t F, int n, int words, int64_t fstride, const uint64_t* __restrict__ bits,
    const uint64_t* __restrict__ bd, const int32_t* __restrict__ A, const int32_t* __restrict__ T,
    const int32_t* __restrict__ M, const int32_t* __restrict__ w,
    const int64_t* __restrict__ row_off, const int64_t* __restrict__ pred_ptr,
    const int32_t* __restrict__ pidx, const int32_t* __restrict__ pdt,
    const int32_t* __restrict__ pdm, const int32_t* __restrict__ pc, int32_t Beff,
    const Cell* __restrict__ m, int64_t T_total, DevStatus* st, int32_t* chain,
    ScheduleOut out) {
  // per-set arrays of small families live in LDS for the whole walk
  __shared__ int32_t s_w[kTraceLds];
  __shared__ int64_t s_off[kTraceLds];
  __shared__ int64_t s_pp[kTraceLds + 1];
  // per chunk of predecessors, alternating by parity: the first hit of each
  // wave and every thread's (source, dt)
  __shared__ int32_t s_first[2][kTraceThreads / kWave];
  __shared__ int32_t s_src[2][kTraceThreads];
  __shared__ int32_t s_dt[2][kTraceThreads];
  __shared__ int32_t s_chain[kMaxNodes + 1];        // a chain adds a node per step
  __shared__ int32_t s_M[kMaxNodes];
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  if (kLds) {
    for (int64_t x = tid; x < F; x += kTraceThreads) {
      s_w[x] = w[x];
      s_off[x] = row_off[x];
      s_pp[x] = pred_ptr[x];
    }
    if (tid == 0) s_pp[F] = pred_ptr[F];
  }
  // Every step of the walk reads the predecessor lists of one set: bring
  // them all into this CU's L2 first when they are small (a few MB), so that
  // those reads cost an L2 hit instead of a trip to memory.
  const int64_t P = pred_ptr[F];
  if (P <= ((int64_t)1 << 17)) {
    int32_t acc = 0;
    for (int64_t x = tid * 16; x < P; x += kTraceThreads * 16)
      acc ^= pidx[x] ^ pdt[x] ^ pc[x] ^ pdm[x];
    if (acc == 0x7fffffff) st->pad0 = acc;          // keeps the loads
  }
  __syncthreads();
  auto Wd = [&](int64_t i) { return kLds ? s_w[i] : w[i]; };
  auto Off = [&](int64_t i) { return kLds ? s_off[i] : row_off[i]; };
  auto PP = [&](int64_t i) { return kLds ? s_pp[i] : pred_ptr[i]; };

  // The walk is identical in every thread; only the predecessor scan is split.
  int64_t j = F - 1;
  int64_t t = st->t_sel;
  int32_t k = 0;
  bool bad = t < 0;
  int par = 0;
  while (j != 0 && !bad) {
    if (t < 0 || t >= Wd(j) || k >= F || k > n) {     // each step removes a node
      bad = true;
      break;
    }
    const int64_t p0 = PP(j), p1 = PP(j + 1);
    const uint32_t mj = m[Off(j) + t];
    int32_t next_i = -1, next_dt = 0;
    for (int64_t base = p0; base < p1 && next_i < 0; base += kTraceThreads) {
      // every load of a chunk is issued unconditionally (a thread past the
      // list reads the list's first pair, a source cell out of its row reads
      // the row's first cell) and the tests come last, so a step waits for
      // the pair data, the source rows' extents and the source cells only
      const int64_t p = base + tid;
      const bool valid = p < p1;
      const int64_t pq = valid ? p : p0;
      const int32_t i = pidx[pq], dt = pdt[pq], c = pc[pq], dm = pdm[pq];
      const int64_t ts = t - dt;
      const bool inrow = valid && ts >= 0 && ts < Wd(i);
      const uint32_t x = m[Off(i) + (inrow ? ts : 0)];
      const bool hit = inrow && x != cell_inf<Cell>() && (int64_t)x <= (int64_t)Beff - c &&
                       (uint32_t)(x + dm) == mj;
      const unsigned long long bal = __ballot(hit);
      if (lane == 0)
        s_first[par][wave] = bal ? wave * kWave + __ffsll((long long)bal) - 1 : INT32_MAX;
      s_src[par][tid] = i;
      s_dt[par][tid] = dt;
      __syncthreads();
      int32_t f = INT32_MAX;
#pragma unroll
      for (int q = 0; q < kTraceThreads / kWave; q++) f = min(f, s_first[par][q]);
      if (f != INT32_MAX) {                    // the smallest predecessor index that hits
        next_i = s_src[par][f];
        next_dt = s_dt[par][f];
      }
      par ^= 1;
    }
    if (next_i < 0 || mj == cell_inf<Cell>()) {
      bad = true;
      break;
    }
    if (tid == 0) chain[k] = (int32_t)j;
    k++;
    t -= next_dt;
    j = next_i;
  }
  if (t != 0) bad = true;                            // the walk must end at (empty, 0)
  __syncthreads();
  finish_schedule<kTraceThreads>(bad ? -1 : k, n, words, fstride, bits, bd, A, T, M, T_total,
                                 chain, out, s_chain, s_M);
}

// The traceback through an optarg slice.  When t* is small, every step of
// the walk stays among the cells (L', t') with t' <= t*: optarg of all of
// them (by the rule of k_trace) is evaluated at once, over the whole chip,
// and the walk then follows it, one load per step instead of a scan of the
// predecessor list.  k_trace_args: workgroup (x, L') takes the 64 cells
// t' = 64 x + lane of row L', its waves the predecessor list in interleaved
// groups of 64 pairs (group g to wave g mod kArgWaves).  Each lane keeps the
// first hit of its wave, and the least over the waves is the first hit of
// the list.  A wave stops when every lane has a hit: its later groups hold
// only larger indices.  The result of cell (L', t') is nxt[L' S + t'] =
// L | (t' - dt) << 16 (S = t* + 1 <= 65536, family indices below 65535), or
// kNoNext: no hit, infinite, L' empty or t' beyond the row.
constexpr int kArgWaves = 4;
constexpr uint32_t kNoNext = 0xFFFFFFFFu;

// The first hit of one wave's share of target j's predecessor list for the
// target cell (j, t) of each lane with value mj (need: the lane has one):
// groups of 64 pairs, every kArgWaves-th from `wave` on.  Returns the index
// in the list, INT32_MAX without a hit.  Every lane of the wave calls it.
template <class Cell>
__device__ __forceinline__ int32_t wave_first_hit(
    int32_t t, uint32_t mj, bool need, int wave, int64_t p0, int64_t p1,
    const int32_t* __restrict__ w, const int64_t* __restrict__ row_off,
    const int32_t* __restrict__ pidx, const int32_t* __restrict__ pdt,
    const int32_t* __restrict__ pdm, const int32_t* __restrict__ pc, int32_t Beff,
    const Cell* __restrict__ m) {
  const int lane = threadIdx.x & (kWave - 1);
  int32_t hit = INT32_MAX;
  if (!__any(need)) return hit;
  for (int64_t g = p0 + (int64_t)wave * kWave; g < p1; g += kArgWaves * kWave) {
    // lane l holds pair g + l: the source row's cell of target t at
    // base + t, in the row when t - dt lies in [0, w_L); past the list w = 0
    const int64_t p = g + lane;
    const int64_t pq = p < p1 ? p : p0;
    const int32_t i = pidx[pq], dt = pdt[pq], c = pc[pq], dm = pdm[pq];
    const int64_t base = row_off[i] - dt;
    const int32_t wi = p < p1 ? w[i] : 0;
    const uint32_t blo = (uint32_t)base, bhi = (uint32_t)((uint64_t)base >> 32);
    const int32_t cnt = (int32_t)std::min<int64_t>(kWave, p1 - g);
    for (int32_t k0 = 0; k0 < cnt; k0 += 8) {
      // eight source cells loaded before any test (a cell outside its row
      // is read at the row's first cell and not used)
      uint32_t x[8];
      bool in[8];
#pragma unroll
      for (int u = 0; u < 8; u++) {
        const int k = k0 + u;
        const int32_t dtk = __builtin_amdgcn_readlane(dt, k);
        const int32_t wk = __builtin_amdgcn_readlane(wi, k);
        const int64_t bk = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane(bhi, k) << 32) |
                                     (uint32_t)__builtin_amdgcn_readlane(blo, k));
        in[u] = (uint32_t)(t - dtk) < (uint32_t)wk;
        x[u] = m[bk + (in[u] ? t : dtk)];
      }
#pragma unroll
      for (int u = 0; u < 8; u++) {
        const int k = k0 + u;
        const int32_t ck = __builtin_amdgcn_readlane(c, k);
        const int32_t dmk = __builtin_amdgcn_readlane(dm, k);
        if (hit == INT32_MAX && in[u] && x[u] != cell_inf<Cell>() &&
            (int64_t)x[u] <= (int64_t)Beff - ck && (uint32_t)(x[u] + dmk) == mj)
          hit = (int32_t)(g - p0) + k;
      }
    }
    if (!__any(need && hit == INT32_MAX)) break;
  }
  return hit;
}

template <class Cell>
__global__ __launch_bounds__(kArgWaves* kWave) void k_trace_args(
    int32_t S, const int32_t* __restrict__ w, const int64_t* __restrict__ row_off,
    const int64_t* __restrict__ pred_ptr, const int32_t* __restrict__ pidx,
    const int32_t* __restrict__ pdt, const int32_t* __restrict__ pdm,
    const int32_t* __restrict__ pc, int32_t Beff, const Cell* __restrict__ m,
    uint32_t* __restrict__ nxt) {
  __shared__ int32_t s_hit[kArgWaves][kWave];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int64_t j = blockIdx.y;
  const int32_t t = blockIdx.x * kWave + lane;
  const int32_t wj = w[j];
  const uint32_t mj = m[row_off[j] + (t < wj ? t : 0)];
  const bool need = j > 0 && t < S && t < wj && mj != cell_inf<Cell>();
  const int64_t p0 = pred_ptr[j], p1 = pred_ptr[j + 1];
  const int32_t hit = wave_first_hit(t, mj, need, wave, p0, p1, w, row_off, pidx, pdt, pdm, pc,
                                     Beff, m);
  s_hit[wave][lane] = need ? hit : INT32_MAX;
  __syncthreads();
  if (wave != 0 || t >= S) return;
  int32_t h = INT32_MAX;
#pragma unroll
  for (int q = 0; q < kArgWaves; q++) h = min(h, s_hit[q][lane]);
  uint32_t e = kNoNext;
  if (h != INT32_MAX) {
    const int64_t p = p0 + h;
    e = (uint32_t)pidx[p] | ((uint32_t)(t - pdt[p]) << 16);
  }
  nxt[j * S + t] = e;
}

// optarg of the whole table where lists are long or the table is small (the
// rule stands at launch_arg_all): 64 cells of target blockIdx.y per
// workgroup, its predecessor list over the workgroup's waves as in
// k_trace_args.
template <class Cell>
__global__ __launch_bounds__(kArgWaves* kWave) void k_arg_split(
    int64_t lb, const int32_t* __restrict__ w, const int64_t* __restrict__ row_off,
    const int64_t* __restrict__ pred_ptr, const int32_t* __restrict__ pidx,
    const int32_t* __restrict__ pdt, const int32_t* __restrict__ pdm,
    const int32_t* __restrict__ pc, int32_t Beff, const Cell* __restrict__ m,
    uint16_t* __restrict__ arg) {
  __shared__ int32_t s_hit[kArgWaves][kWave];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int64_t j = lb + blockIdx.y;
  const int32_t wj = w[j];
  const int32_t t = blockIdx.x * kWave + lane;
  if ((int32_t)(blockIdx.x * kWave) >= wj) return;      // the whole workgroup leaves
  const uint32_t mj = m[row_off[j] + (t < wj ? t : 0)];
  const bool need = j > 0 && t < wj && mj != cell_inf<Cell>();
  const int64_t p0 = pred_ptr[j], p1 = pred_ptr[j + 1];
  s_hit[wave][lane] = wave_first_hit(t, mj, need, wave, p0, p1, w, row_off, pidx, pdt, pdm, pc,
                                     Beff, m);
  __syncthreads();
  if (wave != 0 || t >= wj) return;
  int32_t h = INT32_MAX;
#pragma unroll
  for (int q = 0; q < kArgWaves; q++) h = min(h, s_hit[q][lane]);
  arg[row_off[j] + t] = (uint16_t)(need && h != INT32_MAX ? (uint32_t)pidx[p0 + h] : kNoArg);
}

// The walk over the slice of k_trace_args from (V, t*), then Eq. 1 and
// Eq. 2 of the chain as in k_trace.  Thread 0 walks; meanwhile the other
// waves read the slice from its last row down (the order of the walk), so
// that most of the walk's loads hit the L2 of the XCD it runs on.
__global__ __launch_bounds__(kTraceThreads) void k_trace_follow(
    int64_t F, int n, int words, int64_t fstride, const uint64_t* __restrict__ bits,
    const uint64_t* __restrict__ bd, const int32_t* __restrict__ A, const int32_t* __restrict__ T,
    const int32_t* __restrict__ M, int32_t S, const uint32_t* __restrict__ nxt, int64_t T_total,
    DevStatus* st, int32_t* chain,
    ScheduleOut out) {
  __shared__ int32_t s_chain[kMaxNodes + 1];
  __shared__ int32_t s_M[kMaxNodes];
  __shared__ int32_t s_k;
  const int tid = threadIdx.x;
  if (tid >= kWave) {
    // eight loads in flight per lane
    constexpr int64_t kStride = kTraceThreads - kWave;
    const uint4* q = reinterpret_cast<const uint4*>(nxt);
    uint32_t acc = 0;
    int64_t x = F * S / 4 - 1 - (tid - kWave);
    for (; x >= 7 * kStride; x -= 8 * kStride) {
      uint4 v[8];
#pragma unroll
      for (int u = 0; u < 8; u++) v[u] = q[x - u * kStride];
#pragma unroll
      for (int u = 0; u < 8; u++) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    }
    for (; x >= 0; x -= kStride) {
      const uint4 v = q[x];
      acc ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    if (acc == 0x7fffffffu) st->pad0 = (int32_t)acc;   // keeps the loads
  } else if (tid == 0) {
    int64_t j = F - 1;
    int32_t t = st->t_sel;
    int32_t k = 0;
    bool bad = t < 0 || t >= S;
    while (!bad && j != 0) {
      if (k >= F || k > n) {                      // each step removes a node
        bad = true;
        break;
      }
      const uint32_t e = nxt[j * S + t];
      if (e == kNoNext) {
        bad = true;
        break;
      }
      chain[k++] = (int32_t)j;
      j = e & 0xFFFFu;
      t = (int32_t)(e >> 16);
    }
    if (t != 0) bad = true;                        // the walk must end at (empty, 0)
    s_k = bad ? -1 : k;
  }
  __syncthreads();
  finish_schedule<kTraceThreads>(s_k, n, words, fstride, bits, bd, A, T, M, T_total, chain, out,
                                 s_chain, s_M);
}

}  // namespace

// Launches over all rows, `per` cells of a row to a workgroup, as
// launch(first row, grid): one launch for consecutive levels while their
// longest row leaves at most half of the grid's workgroups without cells.
template <class Launch>
static void for_row_groups(rc_family f, int64_t per, Launch launch) {
  const int64_t L = (int64_t)f->level_ptr.size() - 1;
  for (int64_t l = 0; l < L;) {
    const int64_t first = f->level_ptr[l];
    int64_t most = 0, used = 0, end = l;
    for (; end < L; end++) {
      const int64_t tiles = (f->level_maxw[end] + per - 1) / per;
      const int64_t rows = f->level_ptr[end + 1] - first;
      const int64_t now = used + tiles * (f->level_ptr[end + 1] - f->level_ptr[end]);
      const int64_t wide = std::max(most, tiles);
      if (end > l && wide * rows > 2 * now + 65536) break;
      most = wide;
      used = now;
    }
    launch(first, dim3((unsigned)most, (unsigned)(f->level_ptr[end] - first)));
    l = end;
  }
}

// nb solutions of one family, which agree in cell width and fill.
template <class T>
static void solve_init_t(const rc_solution* sols, int32_t nb, hipStream_t s) {
  rc_family f = sols[0]->f;
  // the row-push and split-panel fills poll cells until they are written
  const int pend = sols[0]->fill_path == 1 || sols[0]->fill_path == 3;
  for (int32_t t0 = 0; t0 < nb; t0 += kTables) {
    InitTables tabs{};
    const int32_t n = std::min<int32_t>(kTables, nb - t0);
    for (int32_t t = 0; t < n; t++) {
      tabs.m[t] = sizeof(T) == 4 ? (void*)sols[t0 + t]->m32 : (void*)sols[t0 + t]->m;
      tabs.st[t] = sols[t0 + t]->status;
      tabs.sentinel[t] = sols[t0 + t]->sentinel;
    }
    auto launch = [&](int64_t lb, dim3 grid) {
      grid.z = (unsigned)n;
      hipLaunchKernelGGL(k_solve_init<T>, grid, dim3(kFillThreads), 0, s, tabs, lb, f->F, f->w,
                         f->row_off, f->cells, sols[0]->objective, pend);
    };
    if (pend)
      for_row_groups(f, kInitChunk, [&](int64_t lb, dim3 grid) {
        grid.x += 1;                                 // a slot is up to kGuard + 63 cells longer
        launch(lb, grid);
      });
    else
      launch(0, dim3(1, (unsigned)f->F));
  }
}

hipError_t launch_solve_init(const rc_solution* sols, int32_t nb, hipStream_t s) {
  for (int32_t a = 0, b; a < nb; a = b) {
    for (b = a + 1; b < nb && sols[b]->cell32 == sols[a]->cell32 &&
                    sols[b]->fill_path == sols[a]->fill_path;)
      b++;
    if (sols[a]->cell32)
      solve_init_t<uint32_t>(sols + a, b - a, s);
    else
      solve_init_t<uint16_t>(sols + a, b - a, s);
  }
  return hipGetLastError();
}

// Waves per workgroup of a level: enough that each walks at most one group
// of the level's longest pair list (1 to 16), but no more than keep eight
// waves per SIMD busy: wide rows already fill the chip with workgroups, and
// their levels are bound by the source reads.  Half or twice these waves
// change a fill by at most 4%.  All levels of a fill, against one round of
// aligned loads and shifts per four pairs (32-bit cells: one thread per
// cell, pair after pair): U-Net 0.58 -> 0.44 ms (4.4 TB/s of source cells),
// ladder40 0.25 -> 0.17, 6199 sets of a 6 x 6 layered graph 3.64 -> 1.67,
// ResNet-50 in 32-bit cells 12.3 -> 1.22.
template <class T>
static void launch_level_vec(rc_family f, int64_t l, int64_t lb, int64_t rows, int32_t Beff, T* m,
                             hipStream_t s) {
  const int64_t tile = kWave * (16 / (int64_t)sizeof(T));
  const dim3 grid((unsigned)((f->level_maxw[l] + tile - 1) / tile), (unsigned)rows);
  const int64_t most = f->level_pairs[l];
  const int64_t blocks = (int64_t)grid.x * grid.y;
  const int64_t cap = 8 * 4 * (int64_t)num_cus();        // eight waves per SIMD
  int nw = 1;
  while (nw < 16 && (int64_t)nw * kLevelGroup < most) nw *= 2;
  while (nw > 1 && blocks * nw > cap) nw /= 2;
#define RCDP_LEVEL_VEC(NW)                                                                   \
  hipLaunchKernelGGL((k_fill_level_vec<T, NW>), grid, dim3(NW * kWave), 0, s, lb, f->w,      \
                     f->row_off, f->pred_ptr, f->lpair, Beff, m)
  switch (nw) {
    case 1: RCDP_LEVEL_VEC(1); break;
    case 2: RCDP_LEVEL_VEC(2); break;
    case 4: RCDP_LEVEL_VEC(4); break;
    case 8: RCDP_LEVEL_VEC(8); break;
    default: RCDP_LEVEL_VEC(16); break;
  }
#undef RCDP_LEVEL_VEC
}

// Source offsets of the vector kernel are 32-bit byte offsets from a row's
// start; longer rows take one cell per thread.
template <class T>
static bool vec_rows(rc_family f) {
  return (f->max_row + 64) * (int64_t)sizeof(T) < INT32_MAX;
}

template <class T>
static void fill_levels(rc_solution sol, T* m, hipStream_t s) {
  rc_family f = sol->f;
  const int64_t L = (int64_t)f->level_ptr.size() - 1;
  for (int64_t l = 1; l < L; l++) {            // level 0 is the empty set
    const int64_t lb = f->level_ptr[l], le = f->level_ptr[l + 1];
    if (le <= lb || f->level_maxw[l] <= 0) continue;
    if (vec_rows<T>(f)) {
      launch_level_vec<T>(f, l, lb, le - lb, (int32_t)sol->Beff, m, s);
    } else {
      const int64_t tiles = ((int64_t)f->level_maxw[l] + kTile - 1) / kTile;
      hipLaunchKernelGGL(k_fill_level<T>, dim3((unsigned)tiles, (unsigned)(le - lb)),
                         dim3(kFillThreads), 0, s, lb, f->w, f->row_off, f->pred_ptr, f->pidx,
                         f->pdt, f->pdm, f->pc, (int32_t)sol->Beff, m);
    }
  }
}

// The family's level-fill pair records, built by its first level fill.
static hipError_t ensure_level_pairs(rc_family f, hipStream_t s) {
  if (f->lpair || f->P == 0) return hipSuccess;
  f->lpair = f->arena.get_n<LevelPair>(f->P);
  if (!f->lpair) return hipErrorOutOfMemory;
  hipLaunchKernelGGL(k_level_pairs, dim3((unsigned)((f->P + 255) / 256)), dim3(256), 0, s, f->P,
                     f->pidx, f->pdt, f->pdm, f->pc, f->w, f->row_off, f->lpair);
  return hipGetLastError();
}

// The halo of every block of the block fill; empty where one leaves a
// workgroup's window or the pair bits were not kept.
void block_fill_halos(rc_family f) {
  f->fb_halo.clear();
  for (int64_t j = 1; j < f->F; j += kFbRows) {
    const auto mm = std::minmax_element(f->w_host.begin() + j,
                                        f->w_host.begin() + std::min<int64_t>(j + kFbRows, f->F));
    const int32_t halo = *mm.second - *mm.first;
    if (halo > kFbHalo) {
      f->fb_halo.clear();
      return;
    }
    f->fb_halo.push_back(halo);
  }
}
int32_t block_fill_rows() { return kFbRows; }

hipError_t launch_fill_block(const rc_solution* sols, int32_t nb, hipStream_t s) {
  rc_family f = sols[0]->f;
  const hipError_t e = ensure_level_pairs(f, s);
  if (e != hipSuccess) return e;
  const int64_t nblk = (int64_t)f->fb_halo.size();
  auto start = [&](int64_t b) { return std::min<int64_t>(1 + b * kFbRows, f->F); };
  auto widest = [&](int64_t a, int64_t b) {
    return b > a ? *std::max_element(f->w_host.begin() + a, f->w_host.begin() + b) : 0;
  };
  for (int32_t t0 = 0; t0 < nb; t0 += kTables) {
    FbTables tabs{};
    const int32_t n = std::min<int32_t>(kTables, nb - t0);
    for (int32_t t = 0; t < n; t++) {
      tabs.m[t] = sols[t0 + t]->m;
      tabs.Beff[t] = (int32_t)sols[t0 + t]->Beff;
    }
    for (int64_t b = 0; b < nblk; b++) {
      FbBlock g{};
      g.j0 = start(b);
      g.j1 = g.n0 = start(b + 1);
      g.n1 = start(b + 2);
      g.halo = f->fb_halo[(size_t)b];
      g.row_blocks = (widest(g.j0, g.j1) + kFbOwn - 1) / kFbOwn;
      constexpr int kTileCells = kWave * 8;
      g.tiles = std::max(1, (widest(g.n0, g.n1) + kTileCells - 1) / kTileCells);
      const dim3 grid((unsigned)(g.row_blocks + (g.n1 - g.n0) * g.tiles), (unsigned)n);
      hipLaunchKernelGGL(k_fill_block, grid, dim3(kFbThreads), 0, s, tabs, g, f->w, f->row_off,
                         f->pred_ptr, f->fb_split, f->pidx, f->pdt, f->pdm, f->pc, f->lpair);
    }
  }
  return hipGetLastError();
}

hipError_t launch_fill(rc_solution sol, hipStream_t s) {
  const hipError_t e = ensure_level_pairs(sol->f, s);
  if (e != hipSuccess) return e;
  if (sol->cell32)
    fill_levels(sol, sol->m32, s);
  else
    fill_levels(sol, sol->m, s);
  return hipGetLastError();
}

hipError_t launch_fronts(rc_solution sol, hipStream_t s) {
  rc_family f = sol->f;
  uint16_t* segmin = sol->arena.get_n<uint16_t>((f->cells >> kSegShift) + f->F + 1);
  if (!segmin) return hipErrorOutOfMemory;
  // a row starts up to 7 cells into its first segment
  auto pass = [&](bool last) {
    for_row_groups(f, kSeg, [&](int64_t lb, dim3 grid) {
      grid.x += 1;
      if (last)
        hipLaunchKernelGGL(k_front, grid, dim3(kFillThreads), 0, s, lb, f->w, f->row_off, sol->m,
                           (const uint16_t*)segmin);
      else
        hipLaunchKernelGGL(k_front_min, grid, dim3(kFillThreads), 0, s, lb, f->w, f->row_off,
                           sol->m, segmin);
    });
  };
  pass(false);
  pass(true);
  return hipGetLastError();
}

template <class T>
static void select_t(const rc_solution* sols, int32_t nb, DevStatus* host, hipStream_t s) {
  rc_family f = sols[0]->f;
  const int64_t v = f->F - 1;
  const int64_t groups = (f->w_host[v] * (int64_t)sizeof(T) + 15) / 16;
  const unsigned blocks = (unsigned)std::max<int64_t>(
      1, std::min<int64_t>((groups + kSelectThreads - 1) / kSelectThreads, kSelectBlocks));
  for (int32_t t0 = 0; t0 < nb; t0 += kTables) {
    SelectTables tabs{};
    const int32_t n = std::min<int32_t>(kTables, nb - t0);
    for (int32_t t = 0; t < n; t++) {
      tabs.m[t] = sizeof(T) == 4 ? (const void*)sols[t0 + t]->m32 : (const void*)sols[t0 + t]->m;
      tabs.st[t] = sols[t0 + t]->status;
    }
    tabs.host = host + t0;
    hipLaunchKernelGGL(k_select<T>, dim3(blocks, (unsigned)n), dim3(kSelectThreads), 0, s, tabs,
                       f->row_off, v, f->w, sols[0]->objective);
  }
}

hipError_t launch_select(const rc_solution* sols, int32_t nb, DevStatus* host, hipStream_t s) {
  for (int32_t a = 0, b; a < nb; a = b) {
    for (b = a + 1; b < nb && sols[b]->cell32 == sols[a]->cell32;) b++;
    if (sols[a]->cell32)
      select_t<uint32_t>(sols + a, b - a, host + a, s);
    else
      select_t<uint16_t>(sols + a, b - a, host + a, s);
  }
  return hipGetLastError();
}

// The slice traceback is taken when its evaluation, about (t* + 1) P pair
// tests spread over the chip, costs less than the longest walk the scan
// could take, and its slice of 4 (t* + 1) F bytes is small; otherwise the
// scan of k_trace.  Measured here: a scan step costs about 0.8 us, the
// slice's tests run at about 5e11 per second (so 4e5 tests per step of the
// longest chain, min(F - 1, n) steps), and its walk costs about 0.2 us a
// step.  RCDP_TRACE = scan | slice forces one (slice within its size limits).
constexpr int64_t kSliceTests = (int64_t)1 << 26;
constexpr int64_t kSliceTestsPerStep = 400000;
constexpr int64_t kSliceCells = (int64_t)1 << 24;

static bool use_slice(rc_solution sol) {
  rc_family f = sol->f;
  const int64_t S = sol->t_star + 1;
  if (sol->t_star < 0 || S > 65536 || f->F >= 65535 || f->F * S > kSliceCells) return false;
  const char* env = std::getenv("RCDP_TRACE");
  if (env && std::strcmp(env, "scan") == 0) return false;
  if (env && std::strcmp(env, "slice") == 0) return true;
  const int64_t steps = std::min<int64_t>(f->F - 1, f->g->n);
  return S * f->P <= std::min<int64_t>(kSliceTests, kSliceTestsPerStep * steps);
}

template <class T>
static hipError_t trace_t(rc_solution sol, const T* m, const ScheduleOut& out, hipStream_t s) {
  rc_family f = sol->f;
  rc_graph g = f->g;
  sol->trace_path = use_slice(sol) ? 1 : 0;
  if (sol->trace_path == 1) {
    const int32_t S = (int32_t)(sol->t_star + 1);
    const int64_t cells = f->F * (int64_t)S;
    if (sol->nxt_cells < cells) {
      sol->nxt = sol->arena.get_n<uint32_t>(cells);
      if (!sol->nxt) return hipErrorOutOfMemory;
      sol->nxt_cells = cells;
    }
    hipLaunchKernelGGL(k_trace_args<T>, dim3((unsigned)((S + kWave - 1) / kWave), (unsigned)f->F),
                       dim3(kArgWaves * kWave), 0, s, S, f->w, f->row_off, f->pred_ptr, f->pidx,
                       f->pdt, f->pdm, f->pc, (int32_t)sol->Beff, m, sol->nxt);
    hipLaunchKernelGGL(k_trace_follow, dim3(1), dim3(kTraceThreads), 0, s, f->F, g->n, g->words,
                       f->fstride, f->bits, f->bd, f->A, g->dT, g->dM, S, sol->nxt, g->T_total,
                       sol->status, sol->chain, out);
  } else if (f->F <= kTraceLds) {
    hipLaunchKernelGGL((k_trace<true, T>), dim3(1), dim3(kTraceThreads), 0, s, f->F, g->n, g->words,
                       f->fstride, f->bits, f->bd, f->A, g->dT, g->dM, f->w, f->row_off,
                       f->pred_ptr, f->pidx, f->pdt, f->pdm, f->pc, (int32_t)sol->Beff, m,
                       g->T_total, sol->status, sol->chain, out);
  } else {
    hipLaunchKernelGGL((k_trace<false, T>), dim3(1), dim3(kTraceThreads), 0, s, f->F, g->n,
                       g->words, f->fstride, f->bits, f->bd, f->A, g->dT, g->dM, f->w,
                       f->row_off, f->pred_ptr, f->pidx, f->pdt, f->pdm, f->pc,
                       (int32_t)sol->Beff, m, g->T_total, sol->status, sol->chain, out);
  }
  return hipGetLastError();
}

hipError_t launch_trace(rc_solution sol, const ScheduleOut& out, hipStream_t s) {
  return sol->cell32 ? trace_t<uint32_t>(sol, sol->m32, out, s)
                     : trace_t<uint16_t>(sol, sol->m, out, s);
}

// optarg of the whole table in as few launches as the rows' lengths allow: no
// cell's optarg depends on another's, so the rows need no order (one launch
// per size level, each waiting for its longest predecessor list, took 5.4 ms
// on resnet50_t10's 167 levels).  A list of at least 64 pairs on average is split over the
// waves of a workgroup, and so are the lists of a table too small to fill
// the chip: there the longest list decides the time.  On long rows with
// short lists (U-Net: 25 pairs, 61 M cells) the extra waves only repeat the
// cells' loads, and one thread per cell is better.  rc_export_table of one
// row, split against one thread per cell: resnet50_t10 57 us against 110,
// densenet121_t10 134 against 265, DenseNet-121 9.7 ms against 16.7,
// ResNet-50 2.2 against 2.9, U-Net 4.8 against 3.2.
constexpr int64_t kSplitCells = (int64_t)1 << 20;

template <class T>
static void arg_all_t(rc_solution sol, const T* m, hipStream_t s) {
  rc_family f = sol->f;
  const bool split = f->P >= kWave * f->F || f->cells <= kSplitCells;
  for_row_groups(f, split ? kWave : kFillThreads, [&](int64_t lb, dim3 grid) {
    if (split)
      hipLaunchKernelGGL(k_arg_split<T>, grid, dim3(kArgWaves * kWave), 0, s, lb, f->w, f->row_off,
                         f->pred_ptr, f->pidx, f->pdt, f->pdm, f->pc, (int32_t)sol->Beff, m,
                         sol->arg);
    else
      hipLaunchKernelGGL(k_arg_all<T>, grid, dim3(kFillThreads), 0, s, lb, f->w, f->row_off,
                         f->pred_ptr, f->pidx, f->pdt, f->pdm, f->pc, (int32_t)sol->Beff, m,
                         sol->arg);
  });
}

hipError_t launch_arg_all(rc_solution sol, hipStream_t s) {
  if (sol->cell32)
    arg_all_t<uint32_t>(sol, sol->m32, s);
  else
    arg_all_t<uint16_t>(sol, sol->m, s);
  return hipGetLastError();
}

}  // namespace rcdp
