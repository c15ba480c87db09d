// Device helpers shared by the kernel sources (inline, header-only).
#pragma once

#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>

#include "katz_internal.h"

namespace katz {

__host__ __device__ inline int bin_of_len(long long len, const BinBounds& bb) {
  return len <= 0 ? BIN_EMPTY
       : len <= bb.g4 ? BIN_G4
       : len <= bb.g8 ? BIN_G8
       : len <= bb.g16 ? BIN_G16
       : len <= bb.g32 ? BIN_G32
       : len <= bb.w16 ? BIN_W16
       : len <= bb.w64 ? BIN_W64
       : len <= kBlockRowMax ? BIN_B256
       : BIN_HUGE;
}


__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

__device__ __forceinline__ unsigned long long lanemask_lt() {
  return (1ull << lane_id()) - 1ull;
}

// Wave-aggregated append: one atomic per wave.  Every lane of the wave must call it.
__device__ __forceinline__ int wave_append(int* counter, bool pred) {
  const unsigned long long mask = __ballot(pred);
  if (mask == 0ull) return -1;
  const int leader = __ffsll((long long)mask) - 1;
  int base = 0;
  if (lane_id() == leader) base = atomicAdd(counter, __popcll(mask));
  base = __shfl(base, leader);
  return base + __popcll(mask & lanemask_lt());
}

// Histogram increment of a wave: h[d] += 1 for every lane with pred.  The
// lanes that share the first active lane's digit add with one LDS atomic (when
// keys share their leading digits, per-lane atomics would queue on one
// address); the others add one by one (spread digits do not collide).  Every
// lane of the wave must call it.
__device__ __forceinline__ void wave_hist_add(unsigned* h, unsigned d, bool pred) {
  const unsigned long long active = __ballot(pred);
  if (!active) return;
  const int leader = __ffsll((long long)active) - 1;
  const unsigned dl = __shfl(d, leader);
  const unsigned long long same = __ballot(pred && d == dl);
  if (lane_id() == leader) atomicAdd(&h[dl], (unsigned)__popcll(same));
  else if (pred && d != dl) atomicAdd(&h[d], 1u);
}

template <bool F32> struct Prec;
template <> struct Prec<false> { using T = double; };
template <> struct Prec<true> { using T = float; };

template <bool F32>
__device__ __forceinline__ typename Prec<F32>::T ldx(const void* x, int32_t j) {
  return reinterpret_cast<const typename Prec<F32>::T*>(x)[j];
}

// ---------------------------------------------------------------------------
// Bound evaluation (Section 3.1, Theorem 1).
//   FP64 form:  l = c + alpha s (undirected) or c;  u = c + beta s.
//   FP32 form:  s = sigma_r x~, with every rounding of the walk vector bounded
//               by the per-node accumulator e and the global factors; the
//               interval [lo, up] contains the exact l_r and u_r.
// ---------------------------------------------------------------------------
// The form is a template argument where several nodes are evaluated per thread:
// a branch on b.fp32 around each would keep their loads from overlapping.
// The bounds of a node from its c, walk entry xv and margin ev (FP32 form).
template <bool F32>
__device__ __forceinline__ void bounds_of(const BoundArgs& b, double cv, typename Prec<F32>::T xv, float ev, double& lo,
                                          double& up) {
  if constexpr (!F32) {
    lo = b.undirected ? cv + b.alpha * xv : cv;
    up = cv + b.beta * xv;
  } else {
    const double s = b.sigma[b.r] * (double)xv;
    const double down = (double)ev * b.f_e + b.tau_coef * b.sigma_sum[b.r];
    const double l = cv * b.f_lo_c + s * b.f_lo_s - down;
    lo = l > 0.0 ? l : 0.0;
    up = cv * b.f_hi_c + down + s * b.f_hi_s;
  }
}

template <bool F32>
__device__ __forceinline__ void bound_eval_as(const BoundArgs& b, int v, double& lo, double& up) {
  bounds_of<F32>(b, b.c[v], reinterpret_cast<const typename Prec<F32>::T*>(b.x)[v], F32 ? b.e[v] : 0.0f, lo, up);
}

__device__ __forceinline__ void bound_eval(const BoundArgs& b, int v, double& lo, double& up) {
  if (b.fp32) bound_eval_as<true>(b, v, lo, up);
  else bound_eval_as<false>(b, v, lo, up);
}

// The bound factors of iteration r of a batched graph (same expressions as the
// host-side bound arguments).
__device__ __forceinline__ void refresh_bounds(BoundArgs& b, const GraphSel& gs, int r) {
  b.r = r;
  b.x = (r & 1) ? gs.xbuf[1] : gs.xbuf[0];
  if (b.fp32) {
    const double u64 = 0x1p-53;
    const double kap = (2.0 * r + 32.0) * u64;
    const double ep = gs.etap[r];
    b.kappa = kap;
    b.f_lo_c = 1.0 - kap;
    b.f_hi_c = 1.0 + kap;
    b.f_e = 1.0 + kap;
    b.f_lo_s = b.undirected ? b.alpha * (1.0 - ep) * (1.0 - kap) * (1.0 - 8.0 * u64) : 0.0;
    b.f_hi_s = b.beta * (1.0 + ep) * (1.0 + kap) * (1.0 + 8.0 * u64);
  }
}

// FP32 form: true while the part of the interval that further iterations
// shrink still exceeds 1/16 of the part they cannot shrink (rounding margin).
template <bool F32>
__device__ __forceinline__ bool can_progress_as(const BoundArgs& b, int v) {
  if constexpr (!F32) return true;
  const double cv = b.c[v];
  const double s = b.sigma[b.r] * (double)reinterpret_cast<const float*>(b.x)[v];
  const double down = (double)b.e[v] * b.f_e + b.tau_coef * b.sigma_sum[b.r];
  const double intrinsic = s * (b.f_hi_s - b.f_lo_s);
  const double margin = 2.0 * down + 2.0 * b.kappa * cv;
  return intrinsic * 16.0 > margin;
}

__device__ __forceinline__ bool can_progress(const BoundArgs& b, int v) {
  return b.fp32 ? can_progress_as<true>(b, v) : true;
}

__device__ __forceinline__ unsigned long long key_of(double lo) {
  return (unsigned long long)__double_as_longlong(lo);
}


// The flags of a run that starts or goes on (M's size and the results stay).
__device__ __forceinline__ void clear_flags(RunScalars* sc) {
  sc->err = 0;
  sc->done = 0;
  sc->status = KATZ_OK;
  sc->top_count = 0;
  sc->kept_count = 0;
  sc->progress = 0;
  sc->cand_count[0] = 0;
  sc->cand_count[1] = 0;
  sc->dmax = 0;
  sc->col_err = 0;
  sc->rescale = 0;
}

// A finished pass's flags to pinned host memory: one 64-bit word, so that the
// host, which polls it, needs no ordering with other stores.  status: -1 while
// the run goes on.  One thread.
__device__ __forceinline__ void publish(const Publish& p, int err, int status, int m, bool many = false) {
  if (!p.to) return;
  __hip_atomic_store(p.to, pass_word(p.seq, err, status, m, many), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Exclusive scan of a long long array of length len with one 1024-thread block.
__device__ inline void block_exclusive_scan_ll(long long* a, long long len, long long* total_out) {
  __shared__ long long wsum[kFinishThreads / kWave];
  __shared__ long long carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  const int t = threadIdx.x;
  const int lane = lane_id();
  const int w = t / kWave;
  for (long long base = 0; base < len; base += kFinishThreads) {
    const long long i = base + t;
    long long x = i < len ? a[i] : 0;
    long long inc = x;
    for (int o = 1; o < kWave; o <<= 1) {
      long long y = __shfl_up(inc, o);
      if (lane >= o) inc += y;
    }
    if (lane == kWave - 1) wsum[w] = inc;
    __syncthreads();
    if (w == 0) {
      long long ws = lane < kFinishThreads / kWave ? wsum[lane] : 0;
      long long wi = ws;
      for (int o = 1; o < kWave; o <<= 1) {
        long long y = __shfl_up(wi, o);
        if (lane >= o) wi += y;
      }
      if (lane < kFinishThreads / kWave) wsum[lane] = wi - ws;   // exclusive wave offsets
    }
    __syncthreads();
    const long long c0 = carry;
    if (i < len) a[i] = c0 + wsum[w] + inc - x;
    __syncthreads();
    if (t == kFinishThreads - 1) carry = c0 + wsum[w] + inc;
    __syncthreads();
  }
  if (t == 0 && total_out) *total_out = carry;
}


// Inside one 1024-thread block: the bucket of hist[0..nb) (nb <= 4096) that holds
// rank `need` (1-based), counting from the largest bucket (desc) or the
// smallest.  Thread t owns positions 4t..4t+3 of that order.
struct Bucket {
  int b;
  int need;   // rank inside the bucket
  int count;  // items in the bucket
};

__device__ inline Bucket find_bucket(const unsigned* h, int nb, int need, bool desc) {
  __shared__ long long wsum[kFinishThreads / kWave];
  __shared__ Bucket res;
  const int t = threadIdx.x;
  const int lane = lane_id();
  const int w = t / kWave;
  unsigned loc[4];
  long long tot = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int pos = 4 * t + j;
    const int bin = desc ? nb - 1 - pos : pos;
    loc[j] = (pos < nb) ? h[bin] : 0u;
    tot += loc[j];
  }
  long long inc = tot;
  for (int o = 1; o < kWave; o <<= 1) {
    long long y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  if (lane == kWave - 1) wsum[w] = inc;
  __syncthreads();
  if (w == 0) {
    long long ws = lane < kFinishThreads / kWave ? wsum[lane] : 0;
    long long wi = ws;
    for (int o = 1; o < kWave; o <<= 1) {
      long long y = __shfl_up(wi, o);
      if (lane >= o) wi += y;
    }
    if (lane < kFinishThreads / kWave) wsum[lane] = wi - ws;
  }
  __syncthreads();
  long long cum = wsum[w] + inc - tot;   // items before this thread's positions
  if (cum < need && need <= cum + tot) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (need <= cum + (long long)loc[j]) {
        const int pos = 4 * t + j;
        res.b = desc ? nb - 1 - pos : pos;
        res.need = (int)(need - cum);
        res.count = (int)loc[j];
        break;
      }
      cum += loc[j];
    }
  }
  __syncthreads();
  const Bucket r = res;
  __syncthreads();
  return r;
}

// Exclusive scan of one int per thread over a 256-thread workgroup; returns the
// thread's prefix and writes the total to *total (all threads).
__device__ inline int block_scan_256(int x, int* total) {
  __shared__ int ws[kWG / kWave];
  const int lane = lane_id();
  const int w = threadIdx.x / kWave;
  int inc = x;
  for (int o = 1; o < kWave; o <<= 1) {
    const int y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  if (lane == kWave - 1) ws[w] = inc;
  __syncthreads();
  int before = 0, all = 0;
  for (int i = 0; i < kWG / kWave; ++i) {
    if (i < w) before += ws[i];
    all += ws[i];
  }
  __syncthreads();
  *total = all;
  return before + inc - x;
}

// Appends for a group of 256 x IPT items (IPT per thread): bit j of `mask` flags
// the thread's j-th item.  One atomic per workgroup reserves the group's slots;
// returns the thread's first slot (its flagged items take consecutive slots).
// Every thread of the workgroup must call it.
__device__ inline int block_reserve(int* counter, unsigned mask) {
  __shared__ int s_base;
  int total = 0;
  const int ex = block_scan_256(__popc(mask), &total);
  if (threadIdx.x == 0) s_base = total > 0 ? atomicAdd(counter, total) : 0;
  __syncthreads();
  const int base = s_base;
  __syncthreads();
  return base + ex;
}

namespace {

// One record per thread: the exchange of the sort's long strides, and (select_small)
// each node's id and upper bound by the slot its record carries.
struct SmallArea {
  unsigned long long key[kFinishThreads];
  int ext[kFinishThreads];
  int slot[kFinishThreads];
  int v[kFinishThreads];   // node id, bit 31: can_progress
  double up[kFinishThreads];
};

// Sorts m <= kFinishThreads records, one per thread (threads at and past m hold
// padding: ~0, INT_MAX), ascending by (key, ext).  Strides below a wave are lane
// exchanges, longer ones go through the LDS: m = 1024 takes 10 of them.  Every
// thread of the workgroup must call it.
__device__ __forceinline__ void sort_records(int m, unsigned long long& key, int& ext, int& slot, SmallArea& sm) {
  const int t = threadIdx.x;
  int P = kWave;
  while (P < m) P <<= 1;
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      unsigned long long ok;
      int oe, os;
      if (stride >= kWave) {
        sm.key[t] = key;
        sm.ext[t] = ext;
        sm.slot[t] = slot;
        __syncthreads();
        ok = sm.key[t ^ stride];
        oe = sm.ext[t ^ stride];
        os = sm.slot[t ^ stride];
        __syncthreads();
      } else {
        ok = __shfl_xor(key, stride);
        oe = __shfl_xor(ext, stride);
        os = __shfl_xor(slot, stride);
      }
      const bool take_min = ((t & stride) == 0) == ((t & size) == 0);
      const bool other_first = ok < key || (ok == key && oe < ext);
      const bool same = ok == key && oe == ext;   // padding records
      if (!same && other_first == take_min) {
        key = ok;
        ext = oe;
        slot = os;
      }
    }
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// Binning, shared by every row source (header-only templates; each kernel source
// instantiates its own copies): prep_count, prep_scan, prep_place.
//
// A workgroup takes kPrepRows rows.  prep_count writes its rows and arcs of each
// class (a bin, or one of SUB parts of a bin by length), its segments of long
// rows and its longest row into one column of a table; prep_scan, one workgroup
// per table row, scans them; prep_place then knows every row's position (class by
// class, rows in their order inside a class) and, from the arcs, where a
// renumbered row starts.  Three launches and two reads of the offsets; bound by
// launches on small graphs (23 launches and two read-backs before, 250 us of a
// call on 2000 nodes) and by the tables written on large ones.
//
// Table rows (of nblocks entries): rows per class, arcs per class, segments,
// longest row; totals holds each row's sum (longest row: maximum).
// ---------------------------------------------------------------------------
namespace {

template <int SUB>
__device__ __forceinline__ int prep_class(long long len, const PrepClasses& pc) {
  const int b = bin_of_len(len, pc.bb);
  if constexpr (SUB == 1) return b;
  int s = 0;
#pragma unroll
  for (int i = 0; i < SUB - 1; ++i) s += len <= pc.sub[b][i] ? 1 : 0;
  return b * SUB + s;
}

template <class Rows, int SUB>
__global__ void __launch_bounds__(kWG) prep_count(Rows rows, long long count, long long* blk, int nblocks,
                                                  RunScalars* sc, PrepClasses pc) {
  constexpr int C = NUM_BINS * SUB;
  constexpr int kPer = kPrepRows / kWG;
  __shared__ int cnt[C];
  __shared__ unsigned long long arcs[C];
  __shared__ int s_seg, s_max, s_rows;
  for (int c = threadIdx.x; c < C; c += kWG) {
    cnt[c] = 0;
    arcs[c] = 0ull;
  }
  if (threadIdx.x == 0) {
    s_seg = 0;
    s_max = 0;
    s_rows = 0;
  }
  __syncthreads();
  const long long base = (long long)blockIdx.x * kPrepRows;
  int dmax = 0, full = 0;   // rows with arcs (the empty ones are what is left)
  bool bad = false;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const long long i = base + j * kWG + threadIdx.x;
    if (i < count) {
      int row;
      long long off, len;
      if (!rows.get(i, row, off, len)) {
        bad = true;
      } else if (len > 0) {
        const int c = prep_class<SUB>(len, pc);
        atomicAdd(&cnt[c], 1);
        atomicAdd(&arcs[c], (unsigned long long)len);
        if (c < SUB) atomicAdd(&s_seg, (int)((len + kSeg - 1) / kSeg));   // BIN_HUGE
        dmax = max(dmax, (int)len);
        ++full;
      }
    }
  }
  if constexpr (Rows::kCsr) {
    if (base == 0 && threadIdx.x == 0 && ((long long)rows.rp[0] != 0 || (long long)rows.rp[count] != rows.nnz))
      bad = true;
  }
  for (int o = 32; o >= 1; o >>= 1) {
    dmax = max(dmax, __shfl_xor(dmax, o));
    full += __shfl_xor(full, o);
  }
  if (lane_id() == 0) {
    atomicMax(&s_max, dmax);
    atomicAdd(&s_rows, full);
  }
  if (bad) atomicOr(&sc->err, 1);
  __syncthreads();
  const int empty = (int)min((long long)kPrepRows, count - base) - s_rows;
  for (int c = threadIdx.x; c < C; c += kWG) {
    blk[(long long)c * nblocks + blockIdx.x] = c == BIN_EMPTY * SUB ? empty : cnt[c];
    blk[(long long)(C + c) * nblocks + blockIdx.x] = (long long)arcs[c];
  }
  if (threadIdx.x == 0) {
    blk[2ll * C * nblocks + blockIdx.x] = s_seg;
    blk[(2ll * C + 1) * nblocks + blockIdx.x] = s_max;
  }
}

// Workgroup i scans table row i (exclusive, in place) and writes its total; the
// last row's is the maximum.  Eight entries per thread and round.
__global__ void __launch_bounds__(kFinishThreads) prep_scan(long long* blk, int nblocks, long long* totals) {
  constexpr int kPer = 8;
  __shared__ long long wsum[kFinishThreads / kWave];
  long long* a = blk + (long long)blockIdx.x * nblocks;
  const bool maximum = blockIdx.x == gridDim.x - 1;
  const int w = threadIdx.x / kWave;
  long long carry = 0;
  for (long long base = 0; base < nblocks; base += kPer * kFinishThreads) {
    const long long i0 = base + (long long)threadIdx.x * kPer;
    long long v[kPer], sum = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      v[j] = i0 + j < nblocks ? a[i0 + j] : 0;
      sum = maximum ? max(sum, v[j]) : sum + v[j];
    }
    long long inc = sum;
    for (int o = 1; o < kWave; o <<= 1) {
      const long long y = __shfl_up(inc, o);
      if (lane_id() >= o) inc = maximum ? max(inc, y) : inc + y;
    }
    __syncthreads();
    if (lane_id() == kWave - 1) wsum[w] = inc;
    __syncthreads();
    long long before = 0, all = 0;
    for (int q = 0; q < kFinishThreads / kWave; ++q) {
      if (q == w) before = all;
      all = maximum ? max(all, wsum[q]) : all + wsum[q];
    }
    if (!maximum) {
      long long run = carry + before + inc - sum;
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        if (i0 + j < nblocks) a[i0 + j] = run;
        run += v[j];
      }
    }
    carry = maximum ? max(carry, all) : carry + all;
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// Descriptors (and segments of long rows) in binned order.  Relabel: the row at
// position p becomes row p of the renumbered graph, its arcs starting where the
// rows before it end; also the tables of both directions.  The first workgroup
// writes the bins' sizes to sc.
template <class Rows, int SUB, bool Relabel>
__global__ void __launch_bounds__(kWG) prep_place(Rows rows, long long count, const long long* blk, int nblocks,
                                                  const long long* totals, RowDesc* desc, SegDesc* segs, HugeRow* huge,
                                                  RunScalars* sc, PrepClasses pc, RelabelOut out) {
  constexpr int C = NUM_BINS * SUB;
  constexpr int kPer = kPrepRows / kWG;
  constexpr int kWaves = kWG / kWave;
  static_assert(C < kWave, "classes are matched by 6 ballots and scanned by one wave");
  if (sc->err) return;
  __shared__ int wcnt[kWaves][C];
  __shared__ int lbase[C + 1];                 // first local place of each class
  __shared__ long long gpos[C], garc[C];       // position and arc offset of the class's first local row
  __shared__ int l_row[kPrepRows], l_len[kPrepRows];
  __shared__ long long l_off[kPrepRows];       // offset in the source; Relabel: then the arcs before the place
  __shared__ uint8_t l_cls[kPrepRows];
  __shared__ int l_seg[kPrepRows];
  __shared__ long long wsum[kWaves];
  const int t = threadIdx.x, lane = lane_id(), w = t / kWave;
  if (blockIdx.x == 0 && t == 0) {
    long long pos = 0;
    for (int b = 0; b < NUM_BINS; ++b) {
      long long n_b = 0;
      for (int s = 0; s < SUB; ++s) n_b += totals[b * SUB + s];
      sc->bin_base[b] = pos;
      sc->bin_count[b] = n_b;
      pos += n_b;
    }
    sc->seg_total = totals[2 * C];
    sc->dmax = (int)totals[2 * C + 1];
  }
  for (int c = lane; c < C; c += kWave) wcnt[w][c] = 0;
  __syncthreads();
  if (w == 0) {
    // Class bases: exclusive scans of the totals over the classes.
    const long long tp = lane < C ? totals[lane] : 0, ta = lane < C ? totals[C + lane] : 0;
    long long ip = tp, ia = ta;
    for (int o = 1; o < kWave; o <<= 1) {
      const long long yp = __shfl_up(ip, o), ya = __shfl_up(ia, o);
      if (lane >= o) {
        ip += yp;
        ia += ya;
      }
    }
    if (lane < C) {
      gpos[lane] = ip - tp + blk[(long long)lane * nblocks + blockIdx.x];
      garc[lane] = ia - ta + blk[(long long)(C + lane) * nblocks + blockIdx.x];
    }
  }
  // Each wave's rows (kPer chunks of 64 consecutive ones): the rank of every row
  // among the wave's rows of its class.
  const long long base = (long long)blockIdx.x * kPrepRows;
  int row[kPer], rank[kPer], cls[kPer];
  long long off[kPer], len[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const long long i = base + w * (kPer * kWave) + j * kWave + lane;
    cls[j] = kWave - 1;   // none
    row[j] = 0;
    off[j] = len[j] = 0;
    if (i < count) {
      rows.get(i, row[j], off[j], len[j]);
      cls[j] = prep_class<SUB>(len[j], pc);
    }
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    unsigned long long peers = ~0ull;
#pragma unroll
    for (int bit = 0; bit < 6; ++bit) {
      const bool on = cls[j] >> bit & 1;
      const unsigned long long m = __ballot(on);
      peers &= on ? m : ~m;
    }
    const int leader = __ffsll((long long)peers) - 1;
    int old = 0;
    if (lane == leader && cls[j] < C) {
      old = wcnt[w][cls[j]];
      wcnt[w][cls[j]] = old + __popcll(peers);
    }
    rank[j] = __shfl(old, leader) + __popcll(peers & lanemask_lt());
  }
  __syncthreads();
  if (w == 0) {
    int tot = 0;
    if (lane < C) {
      for (int q = 0; q < kWaves; ++q) {
        const int c = wcnt[q][lane];
        wcnt[q][lane] = tot;
        tot += c;
      }
    }
    int inc = tot;
    for (int o = 1; o < kWave; o <<= 1) {
      const int y = __shfl_up(inc, o);
      if (lane >= o) inc += y;
    }
    if (lane < C) lbase[lane] = inc - tot;
    if (lane == C) lbase[C] = inc;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    if (cls[j] >= C) continue;
    const int c = cls[j];
    const int in_class = wcnt[w][c] + rank[j];
    const int p = lbase[c] + in_class;
    l_row[p] = row[j];
    l_len[p] = (int)len[j];
    l_off[p] = off[j];
    l_cls[p] = (uint8_t)c;
    if constexpr (Relabel) {
      const int32_t pos = (int32_t)(gpos[c] + in_class);
      out.int_of[row[j]] = pos;
      out.pmap[row[j]] = IdLen{pos, (int32_t)len[j]};
    }
  }
  __syncthreads();
  const int valid = lbase[C];
  // Arcs before each place (four consecutive places per thread).
  long long before[kPer] = {};
  if constexpr (Relabel) {
    long long sum = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      before[j] = sum;
      sum += t * kPer + j < valid ? l_len[t * kPer + j] : 0;
    }
    long long inc = sum;
    for (int o = 1; o < kWave; o <<= 1) {
      const long long y = __shfl_up(inc, o);
      if (lane >= o) inc += y;
    }
    if (lane == kWave - 1) wsum[w] = inc;
    __syncthreads();
    long long start = inc - sum;
    for (int q = 0; q < w; ++q) start += wsum[q];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      // The source offsets leave by position first; then the places take the arcs.
      const int p = q * kWG + t;
      if (p < valid) {
        const int c = l_cls[p];
        const long long pos = gpos[c] + (p - lbase[c]);
        out.ext_of[pos] = l_row[p];
        out.coff[pos] = l_off[p];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j) l_off[t * kPer + j] = start + before[j];
    __syncthreads();
  }
  auto offset_of = [&](int p, int c) {
    if constexpr (Relabel) return garc[c] + l_off[p] - l_off[lbase[c]];
    else return l_off[p];
  };
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int p = q * kWG + t;
    if (p >= valid) break;
    const int c = l_cls[p];
    const long long pos = gpos[c] + (p - lbase[c]);
    desc[pos] = RowDesc{offset_of(p, c), Relabel ? (int32_t)pos : l_row[p], l_len[p]};
  }
  // Rows of more than one segment (their classes come first): the segments
  // before each of them, then one thread per row and one per segment.
  const int n_huge = lbase[SUB];
  if (n_huge == 0) return;
  __syncthreads();
  int nseg[kPer], before_seg = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int p = t * kPer + j;
    nseg[j] = p < n_huge ? (l_len[p] + kSeg - 1) / kSeg : 0;
    before_seg += nseg[j];
  }
  int n_segs = 0;
  int run = block_scan_256(before_seg, &n_segs);
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    l_seg[t * kPer + j] = run;
    run += nseg[j];
  }
  __syncthreads();
  const int part0 = (int)blk[2ll * C * nblocks + blockIdx.x];
  for (int p = t; p < n_huge; p += kWG) {
    const int c = l_cls[p];
    const long long pos = gpos[c] + (p - lbase[c]);
    huge[pos] = HugeRow{Relabel ? (int32_t)pos : l_row[p], l_len[p], (l_len[p] + kSeg - 1) / kSeg, part0 + l_seg[p]};
  }
  for (int q = t; q < n_segs; q += kWG) {
    int lo = 0, hi = n_huge - 1;   // the last row whose segments start at or before q
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (l_seg[mid] <= q) lo = mid;
      else hi = mid - 1;
    }
    const int c = l_cls[lo];
    const int sg = q - l_seg[lo];
    segs[part0 + q] = SegDesc{offset_of(lo, c) + (long long)sg * kSeg, min(kSeg, l_len[lo] - sg * kSeg), part0 + q,
                              (int32_t)(gpos[c] + (lo - lbase[c])), 0};
  }
}

}  // namespace

}  // namespace katz
