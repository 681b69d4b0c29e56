// The smallest feasible budget of a family, on the device.
//
// The experiments of Section 5 run at the smallest budget B for which the
// General Recomputation Problem has a solution, found by binary search.
// Whether B admits a solution does not depend on t: every row minimum of the
// table of Algorithm 1 equals f[L], the same recursion with the t axis taken
// out,
//     f[empty] = 0,   f[L'] = min over L < L' in the family of f[L] + dm(L, L')
//                     over the pairs with f[L] + c(L, L') <= B,
// and B is feasible exactly when f[V] is finite.  Feasibility is monotone
// in B and B = 2 M(V) is always feasible (the one-segment chain {V} peaks at
// 2 M(V)), so the search runs over [0, 2 M(V)].  A round evaluates budgets
// spread over the open interval between the largest budget known infeasible
// and the smallest known feasible, 64 to a workgroup, one per lane, 16 waves
// sharing a target's pairs.  A round runs up to kMbGroups workgroups beside
// each other (fewer where f lies in global scratch), so a range of 2^14
// budgets takes one round and 2^28 two.  Bound by a workgroup's two barriers
// per target, so the rounds decide: ResNet-50 (175 sets, 9365 budgets) 234
// us, where one workgroup, shrinking the interval 65-fold a round, took three
// rounds and 681 us.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rc_internal.h"

namespace rcdp {

namespace {

constexpr int kLanes = 64;
constexpr int kMbRounds = 8;                     // rounds a search can take

// Interval left after a round: lo infeasible, hi feasible.
struct MbRange {
  int32_t lo, hi;
};

typedef const __attribute__((address_space(4))) int32_t cint32;
typedef const __attribute__((address_space(4))) int64_t cint64;

// 64 budgets of a round, one per lane, with f of every set for them ([F][64])
// in LDS when it fits, else in the workgroup's part of global scratch.  The
// pairs of a target are spread over kMbWaves waves: wave w, lane q holds pair
// p0 + kMbWaves q + w of the target (one coalesced load per wave, issued a
// target ahead), every wave relaxes its pairs for the 64 budgets (lane =
// budget, pair values taken with readlane), and the
// waves' partial minima meet in LDS.  Two barriers per target instead of a
// dependent scalar load per pair.
constexpr int kMbWaves = 16;
constexpr int kMbChunk = kMbWaves * kLanes;          // pairs per target and pass

constexpr int kMbGroups = 256;                       // workgroups of a round

template <typename FT, bool kLds>
__global__ __launch_bounds__(kMbChunk) void k_min_budget_waves(int64_t F, int32_t hi0,
                                                                const int64_t* pred_ptr,
                                                                const int32_t* pidx,
                                                                const int32_t* pdm,
                                                                const int32_t* pc, FT* fglob,
                                                                MbRange* range, int round) {
  constexpr FT kInfF = (FT)~(FT)0;                       // every finite f is below it
  extern __shared__ __attribute__((aligned(16))) unsigned char flds_raw[];
  FT* f = kLds ? reinterpret_cast<FT*>(flds_raw)         // [F][64]
               : fglob + (int64_t)blockIdx.x * F * kLanes;
  __shared__ uint32_t red[kMbWaves][kLanes];
  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = threadIdx.x / kLanes;
  cint64* pp = (cint64*)pred_ptr;
  // pair p0 + kMbWaves * lane + wave of target j (j < F), chunk base p0
  auto load = [&](int64_t j, int64_t base, int32_t& i, int32_t& dm, int32_t& c) {
    i = -1;
    dm = 0;
    c = 0;
    if (j >= F) return;
    const int64_t p = base + (int64_t)kMbWaves * lane + wave;
    if (p < pp[j + 1]) {
      i = pidx[p];
      dm = pdm[p];
      c = pc[p];
    }
  };
  // budget x of the round's total (x = 1 .. total) lies x / (total + 1) of the
  // way from the largest infeasible budget to the smallest feasible one
  const int32_t lo = round == 0 ? -1 : range[round - 1].lo;
  const int32_t hi = round == 0 ? hi0 : range[round - 1].hi;
  const int64_t span = (int64_t)hi - lo;
  const int64_t total = (int64_t)gridDim.x * kLanes;
  const int64_t x = (int64_t)blockIdx.x * kLanes + lane + 1;
  const int32_t B = (int32_t)(lo + (x * span + total) / (total + 1));
  if (wave == 0) f[lane] = 0;                            // the empty set
  int32_t ni, ndm, nc;                                   // the next target's first chunk
  load(1, F > 1 ? pp[1] : 0, ni, ndm, nc);
  __syncthreads();
  for (int64_t j = 1; j < F; j++) {
    const int64_t p0 = pp[j], p1 = pp[j + 1];
    int32_t ci = ni, cdm = ndm, cc = nc;
    load(j + 1, j + 1 < F ? pp[j + 1] : 0, ni, ndm, nc);
    uint32_t best = kInfF;
    for (int64_t base = p0; base < p1; base += kMbChunk) {
      if (base != p0) load(j, base, ci, cdm, cc);
      // pairs of this wave in the chunk: base + kMbWaves * q + wave < p1
      const int64_t rem = p1 - base - wave;
      const int nq = rem <= 0 ? 0 : (int)min<int64_t>(kLanes, (rem + kMbWaves - 1) / kMbWaves);
      for (int q = 0; q < nq; q++) {
        const int32_t i = __builtin_amdgcn_readlane(ci, q);
        const int32_t dm = __builtin_amdgcn_readlane(cdm, q);
        const int32_t c = __builtin_amdgcn_readlane(cc, q);
        const uint32_t fi = f[(int64_t)i * kLanes + lane];
        if (fi != kInfF && (int64_t)fi + c <= B) {
          const uint32_t cand = fi + (uint32_t)dm;
          best = cand < best ? cand : best;
        }
      }
    }
    red[wave][lane] = best;
    __syncthreads();
    if (wave == 0) {
      uint32_t m = red[0][lane];
#pragma unroll
      for (int w = 1; w < kMbWaves; w++) m = min(m, red[w][lane]);
      f[j * kLanes + lane] = (FT)m;
    }
    __syncthreads();
  }
  // feasibility is monotone in B: the round's smallest feasible and largest
  // infeasible budgets, over all workgroups
  if (wave != 0) return;
  const bool ok = f[(F - 1) * kLanes + lane] != kInfF;
  int32_t up = ok ? min(B, hi) : hi, down = ok ? lo : max(B, lo);
  for (int off = kLanes / 2; off > 0; off >>= 1) {
    up = min(up, __shfl_xor(up, off, kLanes));
    down = max(down, __shfl_xor(down, off, kLanes));
  }
  if (lane == 0) {
    atomicMin(&range[round].hi, up);
    atomicMax(&range[round].lo, down);
  }
}

__global__ void k_mb_init(int32_t hi0, MbRange* range) {
  if (threadIdx.x < kMbRounds) range[threadIdx.x] = MbRange{-1, hi0};
}

__global__ void k_mb_end(const MbRange* range, int rounds, int32_t hi0, int64_t* out) {
  *out = rounds > 0 ? range[rounds - 1].hi : hi0;
}

}  // namespace

// Value type and home of f: 16 bits when every finite value (at most
// 2 M(V)) fits below the infinity code, LDS when [F][64] fits beside the
// waves' partial minima.
constexpr size_t kMbLds = 60 * 1024;
constexpr size_t kMbHead = 256;                         // the rounds' intervals, the result
static_assert(kMbRounds * sizeof(MbRange) <= kMbHead / 2, "the result lies in the other half");
constexpr size_t kMbScratch = (size_t)32 << 20;         // f in global memory, all workgroups

static int min_budget_kind(rc_family f, int32_t hi0) {
  if (hi0 < 0xFFFF && (size_t)f->F * kLanes * 2 <= kMbLds) return 0;
  if ((size_t)f->F * kLanes * 4 <= kMbLds) return 1;
  return 2;
}

// Workgroups of a round: as many as leave the last budget of the range in
// one round, up to kMbGroups, or to kMbScratch of global memory.
static int64_t min_budget_groups(rc_family f, int32_t hi0, int kind) {
  int64_t most = kMbGroups;
  if (kind == 2)
    most = std::max<int64_t>(1, std::min<int64_t>(64, (int64_t)(kMbScratch / sizeof(uint32_t) /
                                                                kLanes) / f->F));
  return std::min<int64_t>(most, ((int64_t)hi0 + kLanes) / kLanes);
}

size_t min_budget_scratch_bytes(rc_family f, int32_t hi0) {
  const int kind = min_budget_kind(f, hi0);
  size_t bytes = kMbHead;
  if (kind == 2)
    bytes += sizeof(uint32_t) * (size_t)f->F * kLanes * (size_t)min_budget_groups(f, hi0, kind);
  return bytes;
}

hipError_t launch_min_budget(rc_family f, int32_t hi0, void* scratch, int64_t** out,
                             hipStream_t s) {
  const int kind = min_budget_kind(f, hi0);
  const int64_t groups = min_budget_groups(f, hi0, kind);
  MbRange* range = static_cast<MbRange*>(scratch);
  uint32_t* fglob = reinterpret_cast<uint32_t*>(static_cast<char*>(scratch) + kMbHead);
  if (!*out) *out = reinterpret_cast<int64_t*>(static_cast<char*>(scratch) + kMbHead / 2);
  hipLaunchKernelGGL(k_mb_init, dim3(1), dim3(64), 0, s, hi0, range);
  int rounds = 0;
  for (int64_t span = (int64_t)hi0 + 1; span > 1 && rounds < kMbRounds; rounds++) {
    const dim3 grid((unsigned)groups);
    if (kind == 0)
      hipLaunchKernelGGL((k_min_budget_waves<uint16_t, true>), grid, dim3(kMbChunk),
                         sizeof(uint16_t) * (size_t)f->F * kLanes, s, f->F, hi0, f->pred_ptr,
                         f->pidx, f->pdm, f->pc, (uint16_t*)nullptr, range, rounds);
    else if (kind == 1)
      hipLaunchKernelGGL((k_min_budget_waves<uint32_t, true>), grid, dim3(kMbChunk),
                         sizeof(uint32_t) * (size_t)f->F * kLanes, s, f->F, hi0, f->pred_ptr,
                         f->pidx, f->pdm, f->pc, (uint32_t*)nullptr, range, rounds);
    else
      hipLaunchKernelGGL((k_min_budget_waves<uint32_t, false>), grid, dim3(kMbChunk), 0, s, f->F,
                         hi0, f->pred_ptr, f->pidx, f->pdm, f->pc, fglob, range, rounds);
    const int64_t parts = groups * kLanes + 1;
    span = (span + parts - 1) / parts;
  }
  hipLaunchKernelGGL(k_mb_end, dim3(1), dim3(1), 0, s, range, rounds, hi0, *out);
  return hipGetLastError();
}

}  // namespace rcdp
