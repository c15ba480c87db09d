// Stopping criteria of Section 3.1 beyond the LDS-sized top-k test, and the
// separated-pairs measure of Table 1.
//
//   * Top-k with k larger than one workgroup's LDS sort (k > kMaxK), and the
//     ranking criterion, which is the top-k criterion with k = n: after the
//     radix selection and the deactivation pass (sel_apply) the k top nodes
//     are sorted device-wide by (lower bound desc, caller id asc) and every
//     adjacent pair is tested for eps-separation, u(M[i]) - eps < l(M[i-1]).
//   * Score criterion: every node's interval is narrower than eps,
//     u - l < eps; the final list holds every node in ranking order.
//   * Pair criterion: the two given nodes are eps-separated, l(w) > u(v) - eps
//     with w the one ahead by (lower desc, id asc).
//   * Separated pairs (Table 1): the fraction of the n(n-1)/2 unordered pairs
//     {w, v} with l(w) > u(v) or l(v) > u(w); with the lower bounds sorted
//     descending, node v contributes the number of lower bounds above u(v).
//
// The device-wide sort is a merge sort on (key, caller id): 2048-record tiles
// are sorted in LDS by one launch, then each launch merges pairs of sorted runs
// (lk_merge).  What bounds it is launches, not bytes (12 B per record): a sort
// of 5e5 records is 9 launches of 8 to 13 us, where a bitonic network took 45.
//
// The test comes before the sort.  A pair (x, y) of the list with l(x) >= l(y)
// and u(y) - eps >= l(x) fails the test of converged() whether or not other
// nodes lie between the two: y's predecessor p has l(p) <= l(x), so (p, y)
// fails as well.  lk_test sorts each 2048-record tile of the (unsorted) list
// and tests its adjacent pairs; while some tile fails, which is every iteration
// but the last one or two (a renumbered list holds nodes of like degree side by
// side), the device-wide sort does not run; nor does the test while nodes outside the
// top-k survive, which decides the iteration by itself (k = 5000 of a grid of 2^20 nodes,
// 25 passes: 5635 -> 4683 us, with no stop of the host in any of them).
#include <climits>
#include <cstdint>

#include "katz_device.h"

namespace katz {
namespace {

constexpr int kTile = 2 * kFinishThreads;   // records per LDS tile (2048)

__device__ __forceinline__ bool halted(const RunScalars* sc) { return sc->err || sc->done; }
__device__ __forceinline__ int to_ext(const SelArgs& a, int v) { return a.ext_of ? a.ext_of[v] : v; }
__device__ __forceinline__ int to_int(const SelArgs& a, int e) { return a.int_of ? a.int_of[e] : e; }

// A record orders before another when its key is smaller, then its id.  Keys
// are the complemented bit patterns of non-negative lower bounds, so ascending
// keys are descending lower bounds.
__device__ __forceinline__ bool rec_less(unsigned long long ka, int ea, unsigned long long kb, int eb) {
  return ka < kb || (ka == kb && ea < eb);
}

__device__ __forceinline__ void cmp_swap(unsigned long long* key, int32_t* ext, uint16_t* slot, int i, int j) {
  const unsigned long long ki = key[i], kj = key[j];
  const int ei = ext[i], ej = ext[j];
  if (rec_less(kj, ej, ki, ei)) {
    key[i] = kj;
    key[j] = ki;
    ext[i] = ej;
    ext[j] = ei;
    if (slot) {
      const uint16_t s = slot[i];
      slot[i] = slot[j];
      slot[j] = s;
    }
  }
}

// Sorts a tile of kTile records in LDS: a bitonic network in its direction-free
// form (stage s: the mirrored pairs (i, i ^ (s - 1)), then the half-cleaner
// strides s/4 .. 1), one pair per thread and step.
__device__ __forceinline__ void sort_tile(unsigned long long* key, int32_t* ext, uint16_t* slot) {
  const int t = threadIdx.x;
  for (int s = 2; s <= kTile; s <<= 1) {
    const int h = s >> 1;
    const int i0 = (t / h) * s + (t % h);
    cmp_swap(key, ext, slot, i0, i0 ^ (s - 1));
    __syncthreads();
    for (int d = s >> 2; d >= 1; d >>= 1) {
      const int i = (t / d) * 2 * d + (t % d);
      cmp_swap(key, ext, slot, i, i + d);
      __syncthreads();
    }
  }
}

// Bits of RunScalars::fail here: a tile's pair failed (lk_test), a pair of the
// sorted list failed (lk_emit).
constexpr int kTileFail = 2, kPairFail = 1;

// Whether the run stops in this iteration whatever the test says, so that the
// sorted list is the output.
__device__ __forceinline__ bool stops_anyway(const SelArgs& a) {
  const bool walk_zero = a.b.fp32 ? (a.xmax32[a.b.r] == 0u) : (a.xmax64[a.b.r] == 0ull);
  return walk_zero || (a.b.fp32 && !a.sc->progress) || a.b.r >= a.max_iter;
}

// Whether the top list is sorted and tested device-wide in this iteration: no
// node outside the top-k survived and no tile failed, or the run stops here.
__device__ __forceinline__ bool sort_needed(const SelArgs& a) {
  return (a.sc->kept_count == 0 && !(a.sc->fail & kTileFail)) || stops_anyway(a);
}

// The test of the list's tiles (see the head of this file), and the records
// for the sort.  list = null takes the identity list 0..count-1 (k = n, where
// there is no selection: every node is in the list, none is kept beside it).
__global__ void __launch_bounds__(kFinishThreads) lk_test(SelArgs a, const int32_t* list, long long count,
                                                          unsigned long long* key, int32_t* ext) {
  if (halted(a.sc)) return;
  if (list && a.sc->top_count != a.k) {
    // The selection must hand over exactly k top nodes; anything else is an
    // internal inconsistency and stops the run before ids are used.
    if (blockIdx.x == 0 && threadIdx.x == 0) a.sc->err = 2;
    return;
  }
  if (a.sc->kept_count != 0 && !stops_anyway(a)) return;   // (k = n: nothing is kept)
  __shared__ unsigned long long sk[kTile];
  __shared__ int32_t se[kTile];
  __shared__ uint16_t ss[kTile];
  __shared__ double su[kTile];
  const long long base = (long long)blockIdx.x * kTile;
  bool prog = false;
#pragma unroll
  for (int u = 0; u < kTile / kFinishThreads; ++u) {
    const int t = threadIdx.x + u * kFinishThreads;
    const long long i = base + t;
    sk[t] = ~0ull;
    se[t] = INT_MAX;
    ss[t] = (uint16_t)t;
    if (i < count) {
      const int v = list ? list[i] : (int)i;
      double lo, up;
      bound_eval(a.b, v, lo, up);
      const int e = to_ext(a, v);
      key[i] = sk[t] = ~key_of(lo);
      ext[i] = se[t] = e;
      su[t] = up;
      prog = prog || (!list && can_progress(a.b, v));
    }
  }
  __syncthreads();
  sort_tile(sk, se, ss);
  const int valid = (int)min((long long)kTile, count - base);
  bool fail = false;
#pragma unroll
  for (int u = 0; u < kTile / kFinishThreads; ++u) {
    const int t = threadIdx.x + u * kFinishThreads;
    if (t > 0 && t < valid && su[ss[t]] - a.b.eps >= __longlong_as_double((long long)~sk[t - 1])) fail = true;
  }
  const unsigned long long bf = __ballot(fail), bp = __ballot(prog);
  if (lane_id() == 0) {
    if (bf && !(a.sc->fail & kTileFail)) atomicOr(&a.sc->fail, kTileFail);
    if (bp && !a.sc->progress) atomicOr(&a.sc->progress, 1);
  }
}

// sc->need: whether this iteration's list is sorted.  The sort's kernels return at once
// where it is not, given the flags (gate; null: they always run).
__global__ void lk_decide(SelArgs a) {
  if (!halted(a.sc)) a.sc->need = sort_needed(a) ? 1 : 0;
}

__device__ __forceinline__ bool gated_off(const RunScalars* gate) { return gate && (halted(gate) || !gate->need); }

// Sort records of every node (score criterion output): key = ~bits(l), id =
// caller id.
__global__ void __launch_bounds__(kWG) lk_fill(SelArgs a, long long count, unsigned long long* key, int32_t* ext) {
  for (long long i = (long long)blockIdx.x * kWG + threadIdx.x; i < count; i += (long long)gridDim.x * kWG) {
    double lo, up;
    bound_eval(a.b, (int)i, lo, up);
    key[i] = ~key_of(lo);
    ext[i] = to_ext(a, (int)i);
  }
}

// Sorts each tile of the records in place.
__global__ void __launch_bounds__(kFinishThreads) lk_tile(const RunScalars* gate, long long count,
                                                          unsigned long long* key, int32_t* ext) {
  if (gated_off(gate)) return;
  __shared__ unsigned long long sk[kTile];
  __shared__ int32_t se[kTile];
  const long long base = (long long)blockIdx.x * kTile;
  for (int t = threadIdx.x; t < kTile; t += kFinishThreads) {
    const long long i = base + t;
    sk[t] = i < count ? key[i] : ~0ull;
    se[t] = i < count ? ext[i] : INT_MAX;
  }
  __syncthreads();
  sort_tile(sk, se, nullptr);
  for (int t = threadIdx.x; t < kTile; t += kFinishThreads) {
    const long long i = base + t;
    if (i < count) {
      key[i] = sk[t];
      ext[i] = se[t];
    }
  }
}

// How many of the first d records of the merge of a[0..na) and b[0..nb) come
// from a.  One wave searches: every round its 64 lanes test 64 places of the
// remaining range (3 rounds of dependent loads up to 2^18 records, where a
// binary search takes 18).  Every lane of the wave must call it.
__device__ __forceinline__ long long merge_split(const unsigned long long* ka, const int32_t* ea, long long na,
                                                 const unsigned long long* kb, const int32_t* eb, long long nb,
                                                 long long d) {
  long long lo = max(0ll, d - nb), hi = min(d, na);   // the answer is in [lo, hi]
  while (lo < hi) {
    const long long step = (hi - lo + kWave - 1) / kWave;
    const long long i = lo + lane_id() * step;       // is the answer above i?
    bool above = false;
    if (i < hi) {
      // a[i] is among the first d when it orders before b[d - 1 - i].
      const long long j = d - 1 - i;
      above = j >= nb || rec_less(ka[i], ea[i], kb[j], eb[j]);
    }
    const int yes = __popcll(__ballot(above));        // true for a prefix of the lanes
    if (yes == 0) return lo;
    const long long last = lo + (yes - 1) * step;      // the answer is above this place
    hi = min(hi, lo + yes * step);
    lo = last + 1;
  }
  return lo;
}

// One merge pass: sorted runs of `run` records are merged in pairs; a workgroup
// writes 2048 records of the output.  Its two waves of the split search find
// where its share begins and ends in both runs; the share is staged in the LDS,
// where a record's place is its own index plus its rank in the other run.
__global__ void __launch_bounds__(kFinishThreads) lk_merge(const RunScalars* gate, long long count, long long run,
                                                           const unsigned long long* key_in, const int32_t* ext_in,
                                                           unsigned long long* key_out, int32_t* ext_out) {
  if (gated_off(gate)) return;
  __shared__ unsigned long long sk[kTile];
  __shared__ int32_t se[kTile];
  __shared__ long long split[2];
  const long long out0 = (long long)blockIdx.x * kTile;
  const long long pair0 = out0 / (2 * run) * (2 * run);
  const long long na = min(run, count - pair0);
  const long long nb = max(0ll, min(run, count - pair0 - run));
  const unsigned long long* ka = key_in + pair0;
  const int32_t* ea = ext_in + pair0;
  const unsigned long long* kb = ka + na;
  const int32_t* eb = ea + na;
  const long long d0 = out0 - pair0, d1 = min(d0 + kTile, na + nb);
  const int w = threadIdx.x / kWave;
  if (w < 2) {
    const long long s = merge_split(ka, ea, na, kb, eb, nb, w == 0 ? d0 : d1);
    if (lane_id() == 0) split[w] = s;
  }
  __syncthreads();
  const long long a0 = split[0], b0 = d0 - a0;
  const int ca = (int)(split[1] - a0), cb = (int)(d1 - d0) - ca;   // records of the share from a and from b
  for (int t = threadIdx.x; t < ca + cb; t += kFinishThreads) {
    const bool from_a = t < ca;
    sk[t] = from_a ? ka[a0 + t] : kb[b0 + t - ca];
    se[t] = from_a ? ea[a0 + t] : eb[b0 + t - ca];
  }
  __syncthreads();
  for (int t = threadIdx.x; t < ca + cb; t += kFinishThreads) {
    const unsigned long long k = sk[t];
    const int32_t e = se[t];
    // Records of the other part that order before this one.
    int lo = t < ca ? ca : 0, hi = t < ca ? ca + cb : ca;
    const int first = lo;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (rec_less(sk[mid], se[mid], k, e)) lo = mid + 1;
      else hi = mid;
    }
    const long long o = out0 + (t < ca ? t : t - ca) + (lo - first);
    key_out[o] = k;
    ext_out[o] = e;
  }
}

// The sorted list becomes the ranking output; with test = 1 every adjacent
// pair is tested for eps-separation (the check of converged()).
__global__ void __launch_bounds__(kWG) lk_emit(SelArgs a, const RunScalars* gate, long long count, int test,
                                               const unsigned long long* key, const int32_t* ext) {
  if (gated_off(gate)) return;
  bool fail = false;
  for (long long i = (long long)blockIdx.x * kWG + threadIdx.x; i < count; i += (long long)gridDim.x * kWG) {
    const int v = to_int(a, ext[i]);
    double lo, up;
    bound_eval(a.b, v, lo, up);
    a.top_sorted[i] = v;
    a.top_lo[i] = lo;
    a.top_up[i] = up;
    if (test && i > 0 && up - a.b.eps >= __longlong_as_double((long long)~key[i - 1])) fail = true;
  }
  if (test && __ballot(fail) && lane_id() == 0) atomicOr(&a.sc->fail, kPairFail);
}

// converged(), decision: the same rule as the LDS check.
__global__ void lk_finish(SelArgs a) {
  RunScalars* sc = a.sc;
  if (halted(sc)) return;
  const bool walk_zero = a.b.fp32 ? (a.xmax32[a.b.r] == 0u) : (a.xmax64[a.b.r] == 0ull);
  const int kept = sc->kept_count;
  const bool certified = kept == 0 && !sc->fail;
  int status = -1;
  if (certified) status = KATZ_OK;
  else if (walk_zero) status = KATZ_W_EXACT_TIES;
  else if (a.b.fp32 && !sc->progress) status = KATZ_W_PRECISION_LIMIT;
  else if (a.b.r >= a.max_iter) status = KATZ_W_ITER_LIMIT;
  sc->iterations = a.b.r;
  sc->cur = a.act_out_idx;
  sc->m = a.k + kept;
  sc->top_count = 0;
  sc->kept_count = 0;
  sc->cand_count[0] = 0;
  sc->cand_count[1] = 0;
  sc->progress = 0;
  sc->fail = 0;
  if (status >= 0) {
    sc->status = status;
    sc->done = 1;
  }
}

// Score criterion, test: some node has u - l >= eps (fail); FP32 form: some
// such node can still narrow (progress).
__global__ void __launch_bounds__(kWG) score_test(SelArgs a) {
  if (halted(a.sc)) return;
  bool fail = false, prog = false;
  for (long long v = (long long)blockIdx.x * kWG + threadIdx.x; v < a.n; v += (long long)gridDim.x * kWG) {
    double lo, up;
    bound_eval(a.b, (int)v, lo, up);
    if (!(up - lo < a.b.eps)) {
      fail = true;
      if (!prog && can_progress(a.b, (int)v)) prog = true;
    }
  }
  const unsigned long long bf = __ballot(fail), bp = __ballot(prog);
  if (lane_id() == 0) {
    if (bf) atomicOr(&a.sc->fail, 1);
    if (bp) atomicOr(&a.sc->progress, 1);
  }
}

__global__ void score_finish(SelArgs a) {
  RunScalars* sc = a.sc;
  if (halted(sc)) return;
  const bool walk_zero = a.b.fp32 ? (a.xmax32[a.b.r] == 0u) : (a.xmax64[a.b.r] == 0ull);
  int status = -1;
  if (!sc->fail) status = KATZ_OK;
  else if (walk_zero) status = KATZ_W_EXACT_TIES;
  else if (a.b.fp32 && !sc->progress) status = KATZ_W_PRECISION_LIMIT;
  else if (a.b.r >= a.max_iter) status = KATZ_W_ITER_LIMIT;
  sc->iterations = a.b.r;
  sc->m = a.n;
  sc->fail = 0;
  sc->progress = 0;
  if (status >= 0) {
    sc->status = status;
    sc->done = 1;
  }
}

// Pair criterion: test and output (both nodes in ranking order).  ea, eb are
// caller ids.
__global__ void pair_test(SelArgs a, int ea, int eb) {
  RunScalars* sc = a.sc;
  if (halted(sc)) return;
  const int va = to_int(a, ea), vb = to_int(a, eb);
  double la, ua, lb, ub;
  bound_eval(a.b, va, la, ua);
  bound_eval(a.b, vb, lb, ub);
  const bool a_first = la > lb || (la == lb && ea < eb);
  const int w = a_first ? va : vb, v = a_first ? vb : va;
  const double lw = a_first ? la : lb, uw = a_first ? ua : ub;
  const double lv = a_first ? lb : la, uv = a_first ? ub : ua;
  a.top_sorted[0] = w;
  a.top_lo[0] = lw;
  a.top_up[0] = uw;
  a.top_sorted[1] = v;
  a.top_lo[1] = lv;
  a.top_up[1] = uv;
  const bool separated = lw > uv - a.b.eps;
  const bool walk_zero = a.b.fp32 ? (a.xmax32[a.b.r] == 0u) : (a.xmax64[a.b.r] == 0ull);
  int status = -1;
  if (separated) status = KATZ_OK;
  else if (walk_zero) status = KATZ_W_EXACT_TIES;
  else if (a.b.fp32 && !can_progress(a.b, w) && !can_progress(a.b, v)) status = KATZ_W_PRECISION_LIMIT;
  else if (a.b.r >= a.max_iter) status = KATZ_W_ITER_LIMIT;
  sc->iterations = a.b.r;
  sc->m = 2;
  if (status >= 0) {
    sc->status = status;
    sc->done = 1;
  }
}

// Separated pairs: lo holds the n lower bounds in descending order, up the
// upper bounds (any order); adds #{w : lo(w) > up(v)} over v to *count.  Bound
// by the chain of dependent loads of a search per node, so its first steps run
// on every step-th bound, kept in the LDS: 8 dependent loads are left of 19 at
// n = 5e5.
constexpr int kSamples = 2048;

__global__ void __launch_bounds__(kFinishThreads) separated_count(const double* lo, const double* up, long long n,
                                                                  unsigned long long* count) {
  __shared__ double s[kSamples];
  const long long step = (n + kSamples - 1) / kSamples;
  const int ns = (int)((n + step - 1) / step);
  for (int i = threadIdx.x; i < ns; i += kFinishThreads) s[i] = lo[i * step];
  __syncthreads();
  unsigned long long acc = 0;
  for (long long v = (long long)blockIdx.x * kFinishThreads + threadIdx.x; v < n;
       v += (long long)gridDim.x * kFinishThreads) {
    const double u = up[v];
    // First position whose lower bound is not above u (lo is non-increasing).
    int sa = 0, sb = ns;
    while (sa < sb) {
      const int mid = (sa + sb) >> 1;
      if (s[mid] > u) sa = mid + 1;
      else sb = mid;
    }
    // s[sa - 1] is above u, s[sa] is not.
    long long a0 = sa == 0 ? 0 : (sa - 1) * step + 1, b0 = min(n, sa * step);
    while (a0 < b0) {
      const long long mid = a0 + ((b0 - a0) >> 1);
      if (lo[mid] > u) a0 = mid + 1;
      else b0 = mid;
    }
    acc += (unsigned long long)a0;
  }
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o);
  if (lane_id() == 0 && acc) atomicAdd(count, acc);
}

unsigned grid_for(long long items, long long cap) {
  const long long g = (items + kWG - 1) / kWG;
  return (unsigned)std::max<long long>(1, std::min<long long>(g, cap));
}

// Sorts the `count` records in rec[0]; the sorted records end in rec[*which].
hipError_t enqueue_sort(const RunScalars* gate, long long count, const SortRecs rec[2], int* which, hipStream_t s) {
  const unsigned tiles = (unsigned)((count + kTile - 1) / kTile);
  hipLaunchKernelGGL(lk_tile, dim3(tiles), dim3(kFinishThreads), 0, s, gate, count, rec[0].key, rec[0].ext);
  int cur = 0;
  for (long long run = kTile; run < count; run *= 2) {
    hipLaunchKernelGGL(lk_merge, dim3(tiles), dim3(kFinishThreads), 0, s, gate, count, run,
                       (const unsigned long long*)rec[cur].key, (const int32_t*)rec[cur].ext, rec[cur ^ 1].key,
                       rec[cur ^ 1].ext);
    cur ^= 1;
  }
  *which = cur;
  return hipGetLastError();
}

}  // namespace

hipError_t launch_large_test(const SelArgs& a, const SortRecs rec[2], hipStream_t s) {
  const long long k = a.k;
  hipLaunchKernelGGL(lk_test, dim3((unsigned)((k + kTile - 1) / kTile)), dim3(kFinishThreads), 0, s, a,
                     k == a.n ? (const int32_t*)nullptr : (const int32_t*)a.act_out, k, rec[0].key, rec[0].ext);
  hipLaunchKernelGGL(lk_decide, dim3(1), dim3(1), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_large_sort(const SelArgs& a, const SortRecs rec[2], hipStream_t s) {
  int cur = 0;
  const hipError_t e = enqueue_sort(a.sc, a.k, rec, &cur, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(lk_emit, dim3(grid_for(a.k, 1 << 14)), dim3(kWG), 0, s, a, (const RunScalars*)a.sc, (long long)a.k, 1,
                     (const unsigned long long*)rec[cur].key, (const int32_t*)rec[cur].ext);
  return hipGetLastError();
}

hipError_t launch_large_finish(const SelArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(lk_finish, dim3(1), dim3(1), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_score_check(const SelArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(score_test, dim3(grid_for(a.n, 1 << 14)), dim3(kWG), 0, s, a);
  hipLaunchKernelGGL(score_finish, dim3(1), dim3(1), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_score_output(const SelArgs& a, const SortRecs rec[2], hipStream_t s) {
  const long long n = a.n;
  const unsigned g = grid_for(n, 1 << 14);
  hipLaunchKernelGGL(lk_fill, dim3(g), dim3(kWG), 0, s, a, n, rec[0].key, rec[0].ext);
  int cur = 0;
  const hipError_t e = enqueue_sort(nullptr, n, rec, &cur, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(lk_emit, dim3(g), dim3(kWG), 0, s, a, (const RunScalars*)nullptr, n, 0, (const unsigned long long*)rec[cur].key,
                     (const int32_t*)rec[cur].ext);
  return hipGetLastError();
}

hipError_t launch_pair_check(const SelArgs& a, int ea, int eb, hipStream_t s) {
  hipLaunchKernelGGL(pair_test, dim3(1), dim3(1), 0, s, a, ea, eb);
  return hipGetLastError();
}

hipError_t launch_separated_count(const double* lo_desc, const double* up, long long n, unsigned long long* count,
                                  hipStream_t s) {
  hipLaunchKernelGGL(separated_count, dim3(grid_for((n + 3) / 4, 512)), dim3(kFinishThreads), 0, s, lo_desc, up, n, count);
  return hipGetLastError();
}

}  // namespace katz
