// converged() of Algorithm 1 for one graph in one 1024-thread workgroup: the
// radix select of the k-th largest lower bound over M, the deactivation pass
// (u - eps < l(M[k])), the LDS sort of the top-k and the adjacent-pair
// eps-separation test.  A launch handles one graph per workgroup: the batched
// form runs every graph of a batch in one launch, and a single graph uses it
// once its active set is small.
#include <algorithm>

#include "katz_device.h"

namespace katz {
namespace {

constexpr int kSelIlp = 8;   // nodes per thread and pass of the key and deactivation passes

// Positions of the nodes with pred in a list that *counter counts: one atomic per
// wave for all U of a thread (each waits for its return).  Every lane of the wave
// must call it.
template <int U>
__device__ __forceinline__ void wave_append_all(int* counter, const bool (&pred)[U], int (&pos)[U]) {
  unsigned long long mask[U];
  int sum = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    mask[u] = __ballot(pred[u]);
    pos[u] = sum + __popcll(mask[u] & lanemask_lt());
    sum += __popcll(mask[u]);
  }
  if (!sum) return;
  int base = 0;
  if (lane_id() == 0) base = atomicAdd(counter, sum);
  base = __shfl(base, 0);
#pragma unroll
  for (int u = 0; u < U; ++u) pos[u] += base;
}

struct SortArea {
  unsigned long long key[kMaxK];
  int ext[kMaxK];
};

// The end of an iteration's converged(): the status, the size of M, the stop
// flag.  One thread.
template <bool F32>
__device__ __forceinline__ void finish_iteration(RunScalars* sc, const Publish& pub, const BoundArgs& b, int cur, int k,
                                                 int kept, bool failed, bool progress, bool walk_zero, int max_iter) {
  int status = -1;
  if (kept == 0 && !failed) status = KATZ_OK;
  else if (walk_zero) status = KATZ_W_EXACT_TIES;
  else if (F32 && !progress) status = KATZ_W_PRECISION_LIMIT;
  else if (b.r >= max_iter) status = KATZ_W_ITER_LIMIT;
  sc->iterations = b.r;
  sc->cur = cur ^ 1;
  sc->m = k + kept;
  if (status >= 0) {
    sc->status = status;
    sc->done = 1;
  }
  publish(pub, 0, status, k + kept);
}

// converged() for an active set of at most one node per thread: the whole set
// is sorted by (lower desc, id asc), one record per thread, which gives the
// top-k, theta and the pair test at once.  Bound by latency: one round of loads, the sort, one round of stores.  The
// radix digits that larger sets take (below) cost the same for 20 nodes as for
// 20000: on 16 nodes of a graph of 2000, 20.4 -> 6.5 us a launch.
template <bool F32>
__device__ __forceinline__ void select_small(const GraphSel& gs, const Publish& pub, const BoundArgs& b, int cur,
                                             bool identity, int m, bool walk_zero, SmallArea& sm) {
  __shared__ unsigned long long s_theta;
  __shared__ int s_kept, s_fail, s_prog;
  const int32_t* act_in = cur ? gs.act[1] : gs.act[0];
  int32_t* act_out = const_cast<int32_t*>(cur ? gs.act[0] : gs.act[1]);
  const int k = gs.k;
  const int t = threadIdx.x;
  unsigned long long key = ~0ull;   // complemented bits of the lower bound: ascending records
  int ext = INT_MAX;
  int slot = t;
  if (t == 0) {
    s_kept = 0;
    s_fail = 0;
    s_prog = 0;
  }
  if (t < m) {
    const int v = identity ? gs.base + t : act_in[t];
    double lo, up;
    bound_eval_as<F32>(b, v, lo, up);
    key = ~key_of(lo);
    ext = gs.ext_of ? gs.ext_of[v] : v;
    sm.v[t] = v | (can_progress_as<F32>(b, v) ? INT_MIN : 0);
    sm.up[t] = up;
  }
  sort_records(m, key, ext, slot, sm);
  if (t == k - 1) s_theta = ~key;
  sm.key[t] = key;
  __syncthreads();
  if (t < m) {
    const double theta = __longlong_as_double((long long)s_theta);
    const int vp = sm.v[slot];
    const int v = vp & INT_MAX;
    const double up = sm.up[slot];
    const bool top = t < k;
    const bool keep = !top && !(up - b.eps < theta);   // nodes past position k leave M when u - eps < l(M[k])
    if ((top || keep) && vp < 0) s_prog = 1;
    if (top) {
      act_out[t] = v;
      gs.top_sorted[t] = v;
      gs.top_lo[t] = __longlong_as_double((long long)~key);
      gs.top_up[t] = up;
      if (t > 0 && up - b.eps >= __longlong_as_double((long long)~sm.key[t - 1])) s_fail = 1;
    } else if (keep) {
      act_out[k + atomicAdd(&s_kept, 1)] = v;
    }
  }
  __syncthreads();
  if (t == 0) finish_iteration<F32>(gs.sc, pub, b, cur, k, s_kept, s_fail != 0, s_prog != 0, walk_zero, gs.max_iter);
}

// The largest new walk entry over the workgroup maxima of the walk step, into
// xmax[r] (zero before).  Every thread of the workgroup must call it.
template <bool F32>
__device__ __forceinline__ void reduce_walk_max(const GraphSel& gs, const WalkMax& walk) {
  __shared__ double wm[kFinishThreads / kWave];
  double m = 0.0;
  for (int i = threadIdx.x; i < walk.count; i += kFinishThreads)
    m = fmax(m, F32 ? (double)reinterpret_cast<const float*>(walk.blkmax)[i]
                          : reinterpret_cast<const double*>(walk.blkmax)[i]);
  for (int o = 32; o >= 1; o >>= 1) m = fmax(m, __shfl_xor(m, o));
  if (lane_id() == 0) wm[threadIdx.x / kWave] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 0; i < kFinishThreads / kWave; ++i) m = fmax(m, wm[i]);
    if constexpr (F32) const_cast<unsigned*>(gs.xmax32)[gs.b.r] = __float_as_uint((float)m);
    else const_cast<unsigned long long*>(gs.xmax64)[gs.b.r] = (unsigned long long)__double_as_longlong(m);
  }
  __syncthreads();
}

// converged() for up to 16384 nodes (FP32 form: 8192) with the top-k in one record per
// thread: every thread keeps the keys of its nodes in registers.  Above 8192 nodes only
// lists without a floor come here (the first pass of a run in caller order, the re-check
// of an update); those with one are filtered (select_form).  The nodes not behind
// the last of the list's first k are the candidates for the top-k; at most one per
// thread, they are sorted.  More go through radix digits, which read no memory, until
// the k-th key's bucket is that small.  False, with nothing written, when a bucket of
// more records than that carries one key (many ties): the general path resolves those.
// The general path reads and writes every key several times from one workgroup: 16384
// nodes take it 46 us.  On 2000 nodes the digits took 25 us, four places a thread and
// the floor 14.
template <bool F32> constexpr int kMidPer = F32 ? 8 : 16;   // nodes per thread (FP32: more would spill)
template <bool F32> constexpr int kMidActive = kMidPer<F32> * kFinishThreads;
constexpr int kMidIlp = 8;   // nodes whose loads overlap
constexpr int kFinishWaves = kFinishThreads / kWave;

struct MidArea {
  SmallArea rec;
  unsigned h[kDigits];
};

template <bool F32, int kPer>
__device__ __forceinline__ bool select_mid(const GraphSel& gs, const Publish& pub, const BoundArgs& b, int cur,
                                           bool identity, int m, bool walk_zero, MidArea& sm) {
  __shared__ unsigned long long s_kmin, s_kmax, s_theta, s_fkey[kFinishWaves];
  __shared__ int s_fext[kFinishWaves];
  __shared__ unsigned s_place;
  __shared__ int s_cnt, s_cand, s_fail, s_prog, s_cut;
  const int32_t* act_in = cur ? gs.act[1] : gs.act[0];
  int32_t* act_out = const_cast<int32_t*>(cur ? gs.act[0] : gs.act[1]);
  const int32_t* const ext_of = gs.ext_of;
  const int k = gs.k;
  const int t = threadIdx.x;
  if (t == 0) {
    s_kmin = ~0ull;
    s_kmax = 0ull;
    s_cnt = 0;
    s_cand = 0;
    s_place = 0;
    s_fail = 0;
    s_prog = 0;
  }
  __syncthreads();
  unsigned long long key[kPer];
  {
    int node[kPer];   // slots past m hold a valid node that is dropped
    if (identity) {
#pragma unroll
      for (int u = 0; u < kPer; ++u) node[u] = gs.base + (u * kFinishThreads + t < m ? u * kFinishThreads + t : 0);
    } else {
#pragma unroll
      for (int u = 0; u < kPer; ++u) node[u] = act_in[u * kFinishThreads + t < m ? u * kFinishThreads + t : 0];
    }
    const int ext0 = t < k && ext_of ? ext_of[node[0]] : node[0];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      double lo, up;
      bound_eval_as<F32>(b, node[u], lo, up);
      key[u] = key_of(lo);
      if (u % kMidIlp == kMidIlp - 1) __builtin_amdgcn_sched_barrier(0);   // loads in flight, within the registers
    }
    // The last of the list's first k in ranking order (sel_filter's floor: they are
    // the last top-k, or in the first pass of a renumbered run the longest rows).
    unsigned long long fk = t < k ? key[0] : ~0ull;
    int fe = t < k ? ext0 : 0;
    for (int o = 32; o >= 1; o >>= 1) {
      const unsigned long long ok = __shfl_xor(fk, o);
      const int oe = __shfl_xor(fe, o);
      if (ok < fk || (ok == fk && oe > fe)) {
        fk = ok;
        fe = oe;
      }
    }
    if (lane_id() == 0) {
      s_fkey[t / kWave] = fk;
      s_fext[t / kWave] = fe;
    }
  }
  __syncthreads();
  // One bit per node that is not behind the floor.
  unsigned mc = 0;
  {
    unsigned long long fk = s_fkey[lane_id() % kFinishWaves];
    int fe = s_fext[lane_id() % kFinishWaves];
    for (int o = kFinishWaves / 2; o >= 1; o >>= 1) {
      const unsigned long long ok = __shfl_xor(fk, o);
      const int oe = __shfl_xor(fe, o);
      if (ok < fk || (ok == fk && oe > fe)) {
        fk = ok;
        fe = oe;
      }
    }
    int held = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int i = u * kFinishThreads + t;
      bool in = i < m && key[u] > fk;
      if (i < m && key[u] == fk) {
        const int v = identity ? gs.base + i : act_in[i];
        in = (ext_of ? ext_of[v] : v) <= fe;
      }
      mc |= (unsigned)in << u;
      held += __popcll(__ballot(in));
    }
    if (lane_id() == 0 && held) atomicAdd(&s_cand, held);
  }
  __syncthreads();
  const bool floored = s_cand <= kFinishThreads;
  unsigned long long pre = 0;
  int rem = 0, need = k, cnt = s_cand;
  if (!floored) {
    // Too many: radix digits until the k-th key's bucket is small enough.
    unsigned long long kmin = ~0ull, kmax = 0ull;
#pragma unroll
    for (int u = 0; u < kPer; ++u)
      if (u * kFinishThreads + t < m) {
        kmin = key[u] < kmin ? key[u] : kmin;
        kmax = key[u] > kmax ? key[u] : kmax;
      }
    for (int o = 32; o >= 1; o >>= 1) {
      const unsigned long long a = __shfl_xor(kmin, o), c = __shfl_xor(kmax, o);
      kmin = a < kmin ? a : kmin;
      kmax = c > kmax ? c : kmax;
    }
    if (lane_id() == 0) {
      atomicMin(&s_kmin, kmin);
      atomicMax(&s_kmax, kmax);
    }
    __syncthreads();
    const unsigned long long kdiff = s_kmin ^ s_kmax;
    rem = kdiff ? 64 - __clzll((long long)kdiff) : 0;   // low bits still to resolve
    pre = s_kmin >> rem;                                // resolved high bits (keys are below 2^63: rem < 64)
    cnt = m;
    while (cnt > kFinishThreads) {
      if (rem == 0) return false;
      const int w = min(kDigitBits, rem);
      const int shift = rem - w;
      for (int d = t; d < kDigits; d += kFinishThreads) sm.h[d] = 0u;
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kPer; ++u)
        wave_hist_add(sm.h, (unsigned)((key[u] >> shift) & ((1u << w) - 1u)),
                      u * kFinishThreads + t < m && (key[u] >> rem) == pre);
      __syncthreads();
      const Bucket bk = find_bucket(sm.h, 1 << w, need, true);
      pre = (pre << w) | (unsigned)bk.b;
      need = bk.need;
      cnt = bk.count;
      rem = shift;
    }
  }
  // The candidates' or the bucket's records, sorted: the need-th is the last of the top-k.
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int i = u * kFinishThreads + t;
    const bool in = floored ? (mc >> u & 1u) != 0 : i < m && (key[u] >> rem) == pre;
    if (__ballot(in)) {
      const int pos = wave_append(&s_cnt, in);
      if (in) {
        const int v = identity ? gs.base + i : act_in[i];
        sm.rec.key[pos] = ~key[u];
        sm.rec.ext[pos] = ext_of ? ext_of[v] : v;
      }
    }
  }
  __syncthreads();
  {
    unsigned long long rk = t < cnt ? sm.rec.key[t] : ~0ull;
    int re = t < cnt ? sm.rec.ext[t] : INT_MAX, rs = 0;
    __syncthreads();
    sort_records(cnt, rk, re, rs, sm.rec);
    if (t == need - 1) {
      s_theta = ~rk;
      s_cut = re;
    }
  }
  __syncthreads();
  const unsigned long long theta_key = s_theta;
  const double theta = __longlong_as_double((long long)theta_key);
  const int cut = s_cut;
  // Deactivation, from a second evaluation (keeping the upper bounds as well
  // would take more registers than a thread has): one bit per node of the
  // thread for the top-k and one for the others that stay.
  asm volatile("" ::: "memory");   // the bounds are read again, not kept
  unsigned mt = 0, mk = 0;
  bool any = false;
  {
    int node[kPer];
    if (identity) {
#pragma unroll
      for (int u = 0; u < kPer; ++u) node[u] = gs.base + (u * kFinishThreads + t < m ? u * kFinishThreads + t : 0);
    } else {
#pragma unroll
      for (int u = 0; u < kPer; ++u) node[u] = act_in[u * kFinishThreads + t < m ? u * kFinishThreads + t : 0];
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const bool valid = u * kFinishThreads + t < m;
      double lo, up;
      bound_eval_as<F32>(b, node[u], lo, up);
      const bool top = valid && key[u] > theta_key;
      const bool keep = valid && !top && !(up - b.eps < theta);
      mt |= (unsigned)top << u;
      mk |= (unsigned)keep << u;
      if constexpr (F32) any |= (top | keep) & can_progress_as<F32>(b, node[u]);
      if (u % kMidIlp == kMidIlp - 1) __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (!F32) any = true;   // the FP64 form can always go on
    // Nodes tied with the k-th key: the caller ids up to the cut are top.
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      if (u * kFinishThreads + t < m && key[u] == theta_key) {
        const int e = ext_of ? ext_of[node[u]] : node[u];
        if (e <= cut) {
          mt |= 1u << u;
          mk &= ~(1u << u);
          if constexpr (F32) any = any || can_progress_as<F32>(b, node[u]);
        }
      }
    }
  }
  // Places in the new list, in the order of this one: a list in ascending
  // order is read line by line in the next pass, one in any other order takes
  // a line per node (16384 nodes: 50 us a pass).  Counts per 64 nodes (top-k
  // in the low half, others in the high half), scanned by one wave.
  const int w = t / kWave;
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const unsigned c = (unsigned)__popcll(__ballot(mt >> u & 1u)) | (unsigned)__popcll(__ballot(mk >> u & 1u)) << 16;
    if (lane_id() == 0) sm.h[u * kFinishWaves + w] = c;
  }
  __syncthreads();
  if (w == 0) {
    constexpr int kEach = kPer * kFinishWaves / kWave;
    unsigned c[kEach], sum = 0;
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
      c[j] = sum;
      sum += sm.h[lane_id() * kEach + j];
    }
    unsigned inc = sum;
    for (int o = 1; o < kWave; o <<= 1) {
      const unsigned y = __shfl_up(inc, o);
      if (lane_id() >= o) inc += y;
    }
#pragma unroll
    for (int j = 0; j < kEach; ++j) sm.h[lane_id() * kEach + j] = inc - sum + c[j];
    if (lane_id() == kWave - 1) s_place = inc;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const bool top = mt >> u & 1u, keep = mk >> u & 1u;
    const unsigned long long bt = __ballot(top), bk = __ballot(keep);
    const unsigned base = sm.h[u * kFinishWaves + w];
    const int i = u * kFinishThreads + t;
    const int v = top || keep ? (identity ? gs.base + i : act_in[i]) : 0;
    if (top) {
      const int pt = (int)(base & 0xffffu) + __popcll(bt & lanemask_lt());
      if (pt < k) {
        double lo, up;
        bound_eval_as<F32>(b, v, lo, up);
        act_out[pt] = v;
        sm.rec.key[pt] = ~key[u];
        sm.rec.ext[pt] = ext_of ? ext_of[v] : v;
        sm.rec.v[pt] = v;
        sm.rec.up[pt] = up;
      }
    } else if (keep) {
      const int pk = (int)(base >> 16) + __popcll(bk & lanemask_lt());
      if (k + pk < gs.n) act_out[k + pk] = v;
    }
  }
  if (any) s_prog = 1;
  __syncthreads();
  const int kept = (int)(s_place >> 16);
  if ((int)(s_place & 0xffffu) != k) {
    if (t == 0) {
      gs.sc->err = 2;
      publish(pub, 2, -1, 0);
    }
    return true;
  }
  const bool need_sort = kept == 0 || walk_zero || (F32 && !s_prog) || b.r >= gs.max_iter;
  if (need_sort) {
    unsigned long long rk = t < k ? sm.rec.key[t] : ~0ull;
    int re = t < k ? sm.rec.ext[t] : INT_MAX, rs = t;
    __syncthreads();
    sort_records(k, rk, re, rs, sm.rec);
    sm.rec.key[t] = rk;
    __syncthreads();
    if (t < k) {
      const double upv = sm.rec.up[rs];
      gs.top_sorted[t] = sm.rec.v[rs];
      gs.top_lo[t] = __longlong_as_double((long long)~rk);
      gs.top_up[t] = upv;
      if (t > 0 && upv - b.eps >= __longlong_as_double((long long)~sm.rec.key[t - 1])) s_fail = 1;
    }
    __syncthreads();
  }
  if (t == 0) finish_iteration<F32>(gs.sc, pub, b, cur, k, kept, s_fail != 0, s_prog != 0, walk_zero, gs.max_iter);
  return true;
}

// Two kernels share the body, so that each reads its GraphSel from one address
// space (global memory or the kernel arguments) and needs no private copy.
// r: the iteration of a batch (0: one graph, whose arguments hold it).  walk: the
// maxima of the walk step just run, when this launch reduces them itself (one
// graph); null: they are in xmax32 / xmax64.
template <bool F32>
__device__ __forceinline__ void select_graph(const GraphSel& gs, int r, const WalkMax* walk, const Publish& pub) {
  RunScalars* sc = gs.sc;
  if (sc->done || sc->err) {
    if (sc->err && threadIdx.x == 0) publish(pub, sc->err, -1, 0);   // of this pass's walk step
    return;
  }
  if (walk) {
    // Walk step 2 of a renumbered run found a bad column id.
    if (sc->col_err) {
      if (threadIdx.x == 0) {
        sc->err = 1;
        publish(pub, 1, -1, 0);
      }
      return;
    }
    if (walk->blkmax) reduce_walk_max<F32>(gs, *walk);
  }
  BoundArgs b = gs.b;
  if (r) refresh_bounds(b, gs, r);
  const int cur = r ? sc->cur : gs.cur;
  const int32_t* act_in = cur ? gs.act[1] : gs.act[0];
  int32_t* act_out = const_cast<int32_t*>(cur ? gs.act[0] : gs.act[1]);
  const bool identity = !r && gs.identity_in;
  const int m = identity ? gs.n : sc->m;
  const bool walk_zero = F32 ? (gs.xmax32[b.r] == 0u) : (gs.xmax64[b.r] == 0ull);
  __shared__ union {
    unsigned h[kDigits];
    SortArea srt;
    SmallArea small;
    MidArea mid;
  } sm;
  if (m <= kFinishThreads) {
    select_small<F32>(gs, pub, b, cur, identity, m, walk_zero, sm.small);
    return;
  }
  if (walk && gs.k <= kFinishThreads) {
    if (m <= 4 * kFinishThreads) {
      if (select_mid<F32, 4>(gs, pub, b, cur, identity, m, walk_zero, sm.mid)) return;
    } else if (m <= kMidActive<F32>) {
      if (select_mid<F32, kMidPer<F32>>(gs, pub, b, cur, identity, m, walk_zero, sm.mid)) return;
    }
  }
  const int k = gs.k;
  // The graph's arrays and sizes as locals: read from gs once, not again after
  // every store (gs may sit in global memory, which the stores could alias).
  const int base_id = gs.base;
  const int n_g = gs.n;
  unsigned long long* const keys = gs.keys;
  unsigned long long* const cand_key = gs.cand_key;
  int32_t* const cand_v = gs.cand_v;
  const int32_t* const ext_of = gs.ext_of;
  const int32_t* const int_of = gs.int_of;
  int32_t* const top_sorted = gs.top_sorted;
  double* const top_lo = gs.top_lo;
  double* const top_up = gs.top_up;
  auto ext = [ext_of](int v) { return ext_of ? ext_of[v] : v; };
  const int t = threadIdx.x;

  __shared__ unsigned long long s_prefix, s_kmin, s_kmax;
  __shared__ int s_need, s_count, s_cnt, s_top, s_kept, s_fail, s_prog, s_idpre, s_idneed;

  // Keys of M, with their minimum and maximum: the bits above the highest bit
  // in which two keys differ are common to all keys, so the radix digits start
  // right below them (the keys of one graph often share their exponent, and a
  // digit inside it would leave every node a candidate).  Every digit choice
  // finds the same k-th key.
  if (t == 0) {
    s_cnt = 0;
    s_top = 0;
    s_kept = 0;
    s_fail = 0;
    s_prog = 0;
    s_kmin = ~0ull;
    s_kmax = 0ull;
  }
  __syncthreads();
  {
    unsigned long long kmin = ~0ull, kmax = 0ull;
    // kSelIlp nodes per thread and pass, their loads issued together (a slot past
    // the end evaluates node base, a valid index, and is dropped).
    for (int b0 = 0; b0 < m; b0 += kSelIlp * kFinishThreads) {   // same trip count for every thread
      unsigned long long kk[kSelIlp];
#pragma unroll
      for (int u = 0; u < kSelIlp; ++u) {
        const int i = b0 + u * kFinishThreads + t;
        const int v = i < m ? (identity ? base_id + i : act_in[i]) : base_id;
        double lo, up;
        bound_eval_as<F32>(b, v, lo, up);
        kk[u] = key_of(lo);
      }
#pragma unroll
      for (int u = 0; u < kSelIlp; ++u) {
        const int i = b0 + u * kFinishThreads + t;
        if (i < m) {
          keys[i] = kk[u];
          kmin = kk[u] < kmin ? kk[u] : kmin;
          kmax = kk[u] > kmax ? kk[u] : kmax;
        }
      }
    }
    for (int o = 32; o >= 1; o >>= 1) {
      const unsigned long long a = __shfl_xor(kmin, o), c = __shfl_xor(kmax, o);
      kmin = a < kmin ? a : kmin;
      kmax = c > kmax ? c : kmax;
    }
    if (lane_id() == 0) {
      atomicMin(&s_kmin, kmin);
      atomicMax(&s_kmax, kmax);
    }
  }
  __syncthreads();
  const unsigned long long kdiff = s_kmin ^ s_kmax;
  int rem = kdiff ? 64 - __clzll((long long)kdiff) : 0;   // low bits still to resolve
  if (rem > 63) rem = 63;                                   // keys of non-negative bounds are below 2^63
  unsigned long long pre = m > 0 ? (s_kmin >> rem) : 0ull;  // resolved high bits of the k-th key
  // Level 0 over M: histogram of the first digit below the common bits, then
  // the candidates, the nodes in the k-th key's bucket.
  {
    const int w = min(kDigitBits, rem);
    const int shift = rem - w;
    for (int d = t; d < kDigits; d += kFinishThreads) sm.h[d] = 0u;
    __syncthreads();
    for (int b0 = 0; b0 < m; b0 += kSelIlp * kFinishThreads) {
      unsigned long long kk[kSelIlp];
#pragma unroll
      for (int u = 0; u < kSelIlp; ++u) {
        const int i = b0 + u * kFinishThreads + t;
        kk[u] = i < m ? keys[i] : 0ull;
      }
#pragma unroll
      for (int u = 0; u < kSelIlp; ++u)
        wave_hist_add(sm.h, (unsigned)((kk[u] >> shift) & ((1u << w) - 1u)), b0 + u * kFinishThreads + t < m);
    }
    __syncthreads();
    const Bucket bk = find_bucket(sm.h, 1 << w, k, true);
    if (t == 0) {
      s_prefix = (pre << w) | (unsigned)bk.b;
      s_need = bk.need;
      s_count = bk.count;
    }
    __syncthreads();
    pre = s_prefix;
    rem = shift;
    for (int b0 = 0; b0 < m; b0 += kSelIlp * kFinishThreads) {
      unsigned long long kk[kSelIlp];
      int vv[kSelIlp];
#pragma unroll
      for (int u = 0; u < kSelIlp; ++u) {
        const int i = b0 + u * kFinishThreads + t;
        kk[u] = i < m ? keys[i] : 0ull;
        vv[u] = i < m ? (identity ? base_id + i : act_in[i]) : 0;
      }
      bool pred[kSelIlp];
      int pos[kSelIlp];
#pragma unroll
      for (int u = 0; u < kSelIlp; ++u) pred[u] = b0 + u * kFinishThreads + t < m && (kk[u] >> rem) == pre;
      wave_append_all(&s_cnt, pred, pos);
#pragma unroll
      for (int u = 0; u < kSelIlp; ++u)
        if (pred[u]) {
          cand_key[pos[u]] = kk[u];
          cand_v[pos[u]] = vv[u];
        }
    }
  }
  __syncthreads();
  const int cnt = s_cnt;
  // Remaining digits over the candidates, at most 12 bits each.
  while (rem > 0) {
    const int w = min(kDigitBits, rem);
    const int shift = rem - w;
    for (int d = t; d < kDigits; d += kFinishThreads) sm.h[d] = 0u;
    __syncthreads();
    for (int i0 = 0; i0 < cnt; i0 += kSelIlp * kFinishThreads) {
      unsigned long long kk[kSelIlp];
#pragma unroll
      for (int u = 0; u < kSelIlp; ++u) {
        const int i = i0 + u * kFinishThreads + t;
        kk[u] = i < cnt ? cand_key[i] : 0ull;
      }
#pragma unroll
      for (int u = 0; u < kSelIlp; ++u) {
        const int i = i0 + u * kFinishThreads + t;
        wave_hist_add(sm.h, (unsigned)((kk[u] >> shift) & ((1u << w) - 1u)), i < cnt && (kk[u] >> rem) == pre);
      }
    }
    __syncthreads();
    const Bucket bk = find_bucket(sm.h, 1 << w, s_need, true);
    if (t == 0) {
      s_prefix = (pre << w) | (unsigned)bk.b;
      s_need = bk.need;
      s_count = bk.count;
    }
    __syncthreads();
    pre = s_prefix;
    rem = shift;
  }
  const unsigned long long theta_key = s_prefix;
  const double theta = __longlong_as_double((long long)theta_key);
  const int need = s_need;
  const int ties = s_count;
  int cut = INT_MAX;
  if (need < ties) {
    // The need-th smallest id among the ties (ids are 31-bit: 11 + 11 + 9 bits).
    if (t == 0) {
      s_idpre = 0;
      s_idneed = need;
    }
    __syncthreads();
    int shift = 31;
    for (int L = 0; L < 3; ++L) {
      const int width = L < 2 ? 11 : 9;
      const int hishift = shift;
      shift -= width;
      for (int d = t; d < kDigits; d += kFinishThreads) sm.h[d] = 0u;
      __syncthreads();
      const int idpre = s_idpre;
      // Tied ids share their high digits (all of them at the first level when
      // the ids are below 2^20), so the counts go through the wave-aggregated
      // add; the loop has the same trip count for every thread.
      for (int i0 = 0; i0 < cnt; i0 += kFinishThreads) {
        const int i = i0 + t;
        const bool tie = i < cnt && cand_key[i] == theta_key;
        const int e = tie ? ext(cand_v[i]) : 0;
        const bool in = tie && (hishift >= 31 ? 0 : (e >> hishift)) == idpre;
        wave_hist_add(sm.h, (unsigned)((e >> shift) & ((1 << width) - 1)), in);
      }
      __syncthreads();
      const Bucket ib = find_bucket(sm.h, 1 << width, s_idneed, false);
      if (t == 0) {
        s_idpre = (idpre << width) | ib.b;
        s_idneed = ib.need;
      }
      __syncthreads();
    }
    cut = s_idpre;
  }
  // Deactivation: nodes past position k leave M when u - eps < l(M[k]).
  // kSelIlp nodes per thread and pass as above (the order of M does not matter).
  {
    bool prog = false;
    for (int base = 0; base < m; base += kSelIlp * kFinishThreads) {
      bool top[kSelIlp], keep[kSelIlp];
      int vv[kSelIlp];
#pragma unroll
      for (int u = 0; u < kSelIlp; ++u) {
        const int i = base + u * kFinishThreads + t;
        const bool valid = i < m;
        const int v = valid ? (identity ? base_id + i : act_in[i]) : base_id;
        const unsigned long long key = valid ? keys[i] : 0ull;
        double lo, up;
        bound_eval_as<F32>(b, v, lo, up);
        top[u] = valid && (key > theta_key || (key == theta_key && ext(v) <= cut));
        keep[u] = valid && !top[u] && !(up - b.eps < theta);
        if ((top[u] || keep[u]) && can_progress_as<F32>(b, v)) prog = true;
        vv[u] = v;
      }
      int pt[kSelIlp], pk[kSelIlp];
      wave_append_all(&s_top, top, pt);
      wave_append_all(&s_kept, keep, pk);
#pragma unroll
      for (int u = 0; u < kSelIlp; ++u) {
        if (top[u] && pt[u] < k) act_out[pt[u]] = vv[u];
        if (keep[u] && k + pk[u] < n_g) act_out[k + pk[u]] = vv[u];
      }
    }
    if (prog) s_prog = 1;
  }
  __syncthreads();
  if (s_top != k) {
    if (t == 0) {
      sc->err = 2;
      publish(pub, 2, -1, 0);
    }
    return;
  }
  // Sort the top-k by (lower desc, id asc) and test adjacent pairs: needed when
  // no node outside the top-k survived, or as the output when the run stops
  // here for another reason.
  const bool need_sort = s_kept == 0 || walk_zero || (F32 && !s_prog) || b.r >= gs.max_iter;
  int P = 1;
  while (P < k) P <<= 1;
  if (!need_sort) P = 0;
  if (t == 0 && !need_sort) s_fail = 1;
  for (int i = t; i < P; i += kFinishThreads) {
    if (i < k) {
      const int v = act_out[i];
      double lo, up;
      bound_eval_as<F32>(b, v, lo, up);
      sm.srt.key[i] = key_of(lo);
      sm.srt.ext[i] = ext(v);
    } else {
      sm.srt.key[i] = 0ull;
      sm.srt.ext[i] = INT_MAX;
    }
  }
  __syncthreads();
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int q = t; q < P / 2; q += kFinishThreads) {
        const int i = 2 * q - (q & (stride - 1));
        const int j = i + stride;
        const bool up = ((i & size) == 0);
        const unsigned long long ki = sm.srt.key[i], kj = sm.srt.key[j];
        const int ei = sm.srt.ext[i], ej = sm.srt.ext[j];
        const bool j_before_i = kj > ki || (kj == ki && ej < ei);
        if (j_before_i == up) {
          sm.srt.key[i] = kj;
          sm.srt.key[j] = ki;
          sm.srt.ext[i] = ej;
          sm.srt.ext[j] = ei;
        }
      }
      __syncthreads();
    }
  }
  for (int i = t; i < (need_sort ? k : 0); i += kFinishThreads) {
    const int v = int_of ? int_of[sm.srt.ext[i]] : sm.srt.ext[i];
    double lo, up;
    bound_eval_as<F32>(b, v, lo, up);
    top_sorted[i] = v;
    top_lo[i] = lo;
    top_up[i] = up;
    if (i > 0 && up - b.eps >= __longlong_as_double((long long)sm.srt.key[i - 1])) s_fail = 1;
  }
  __syncthreads();
  if (t == 0) finish_iteration<F32>(sc, pub, b, cur, k, s_kept, s_fail != 0, s_prog != 0, walk_zero, gs.max_iter);
}

// One workgroup per graph; then, while the graph goes on, what its next iteration
// needs: the FP32 scale 2^e above deg_max * max(x~_r) and the rounding bound
// eta_{r+1} (the host's recurrences), and a cleared maximum.
template <bool F32>
__global__ void __launch_bounds__(kFinishThreads) select_wg(const GraphSel* gsel, int r, BatchNext nx) {
  const int g = blockIdx.x;
  RunScalars* sc = gsel[g].sc;
  if (sc->done || sc->err) return;
  select_graph<F32>(gsel[g], r, nullptr, Publish{nullptr, 0});
  if (threadIdx.x != 0) return;
  if (sc->done || sc->err) {   // written by this thread
    atomicAdd(nx.ndone, 1);
    return;
  }
  if (r + 1 >= nx.stride) return;
  const long long at = (long long)g * nx.stride;
  nx.gxmax32[at + r + 1] = 0u;
  nx.gxmax64[at + r + 1] = 0ull;
  if constexpr (F32) {
    const float M = __uint_as_float(nx.gxmax32[at + r]);
    int ex = 0;
    if (M > 0.0f) {
      (void)frexpf(M, &ex);
      ex += nx.gclog2[g];
    }
    const double sg = ldexp(nx.galpha[g] * nx.gsigma[at + r], ex);
    nx.gexp[at + r + 1] = ex;
    nx.gsigma[at + r + 1] = sg;
    nx.gsigsum[at + r + 1] = nx.gsigsum[at + r] + sg;
    const double eta = ((1.0 + nx.eta[at + r]) * (1.0 + nx.grho[g]) - 1.0) * (1.0 + 0x1p-50);
    nx.eta[at + r + 1] = eta;
    nx.etap[at + r + 1] = eta / (1.0 - eta) * (1.0 + 0x1p-50);
  }
}

template <bool F32>
__global__ void __launch_bounds__(kFinishThreads) select_wg_one(GraphSel one, WalkMax walk, Publish pub) {
  select_graph<F32>(one, 0, &walk, pub);
}

}  // namespace

hipError_t launch_select_wg(const GraphSel* gsel, int count, int r, int fp32, const BatchNext& next, hipStream_t s) {
  if (count > 0) {
    if (fp32) hipLaunchKernelGGL(select_wg<true>, dim3(count), dim3(kFinishThreads), 0, s, gsel, r, next);
    else hipLaunchKernelGGL(select_wg<false>, dim3(count), dim3(kFinishThreads), 0, s, gsel, r, next);
  }
  return hipGetLastError();
}

hipError_t launch_select_wg_one(const GraphSel& one, const WalkMax& walk, const Publish& pub, hipStream_t s) {
  if (one.b.fp32) hipLaunchKernelGGL(select_wg_one<true>, dim3(1), dim3(kFinishThreads), 0, s, one, walk, pub);
  else hipLaunchKernelGGL(select_wg_one<false>, dim3(1), dim3(kFinishThreads), 0, s, one, walk, pub);
  return hipGetLastError();
}

}  // namespace katz
