// PageRank by power iteration in double precision (Table I's PR primitive;
// the rank update and the accumulation over edges of Alg. 3), on an
// undirected CSR where every edge carries rank both ways.
//
// rank_0(v) = 1/n.  Iteration i reads contrib_i(u) = rank_i(u) / deg(u) and
// writes, for every vertex v,
//   acc(v)         = sum over the neighbours u of v of contrib_i(u)
//   rank_{i+1}(v)  = (1 - d)/n + d acc(v)
//   contrib_{i+1}(v) = rank_{i+1}(v) / deg(v)   (0 for degree 0)
// in one pass: the accumulation is a gather over v's own row (a pull, no
// atomics), so each vertex's new rank is final when its row is done.
// Convergence (the threshold ratio): the run stops after an iteration in
// which every vertex changed by at most tol times its previous rank; tol = 0
// runs max_iter iterations.  The host enqueues everything without reading
// back: an iteration is a launch that returns at once when the run has already
// stopped, or all are one launch that ends there.
//
// Two forms.  The planned one renumbers the vertices by falling degree at the
// start of the call and copies the columns once under the new numbers: the
// contributions most entries ask for then lie together, rows of one length
// are neighbours, and each class of rows gets the lanes that fit it.  The
// direct one works on the CSR arrays as they are; it is taken for too few
// iterations to pay for the plan and where the workspace has no room for the
// copied columns.  Every row's sum is formed in a fixed
// order in both, so ranks do not change from call to call.
//
// What bounds it (R-MAT 22, 128 M entries, 20 iterations): gathers that miss
// the LDS and the L1 cost one L2 request each, and the L2s together serve
// about 110 G random ones a second.  The direct form's iteration takes
// 1285 us (work counter 190 us, nearly every gather a request); renumbered
// and with rows in classes 840 us; with the first 18 k contributions in LDS
// 677 us (78 M requests); with the long rows' columns split over the XCDs
// 415 us (pp_long 298 us for 32 M requests, pp_iter 116 us).  The plan costs
// 1.86 ms, 1.75 ms of it the 125 M requests for the columns' new numbers.
// The call: 25.6 -> 10.2 ms; n = 20,000, 12 iterations: 1534 -> 280 us.
#include <math.h>
#include <string.h>

#include "fg_common.h"
#include "frontier.h"

namespace {

constexpr int PR_BT = 256;
constexpr int PR_LONG = 4096;  // rows at least this long are summed by a workgroup

struct PrCtl {
  uint32_t next_item[2];  // work counters, slot = iteration parity
  uint32_t blocks_done;
  int32_t nlong;          // rows of at least PR_LONG entries
  int32_t done;           // converged (tol > 0)
  int32_t iterations;
  unsigned long long notconv[2];  // vertices above the threshold, slot = parity
};

struct PrArgs {
  int32_t n;
  int64_t m;
  const int32_t* off;
  const int32_t* col;
  double d;      // damping
  double base;   // (1 - d) / n
  double tol;
  double* rank;
  double* contrib[2];
  int32_t* longrows;
  PrCtl* ctl;
  fg_run_stats* stats;
  int32_t clock_khz;
};

__device__ __forceinline__ double wave_sum_f64(double x) {
#pragma unroll
  for (int s = FG_WAVE / 2; s > 0; s >>= 1) x += __shfl_xor(x, s, FG_WAVE);
  return x;
}

// The update of one vertex from its accumulated sum (no contraction into
// fused multiply-adds: the products and sums round as written).
__device__ __forceinline__ unsigned long long pr_update(const PrArgs& A, double* nxt, int32_t v,
                                                        int32_t deg, double acc) {
  const double nr = __dadd_rn(A.base, __dmul_rn(A.d, acc));
  const double old = A.rank[v];
  const double diff = nr > old ? __dsub_rn(nr, old) : __dsub_rn(old, nr);
  A.rank[v] = nr;
  nxt[v] = deg > 0 ? nr / (double)deg : 0.0;
  return diff > __dmul_rn(A.tol, old) ? 1ull : 0ull;
}

__global__ __launch_bounds__(PR_BT) void pr_setup_kernel(PrArgs A, double inv_n) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nth = (int64_t)gridDim.x * blockDim.x;
  for (int64_t v = tid; v < A.n; v += nth) {
    const int32_t deg = A.off[v + 1] - A.off[v];
    A.rank[v] = inv_n;
    A.contrib[0][v] = deg > 0 ? inv_n / (double)deg : 0.0;
    if (deg >= PR_LONG) A.longrows[atomicAdd(&A.ctl->nlong, 1)] = (int32_t)v;
  }
  if (tid == 0 && A.stats) {
    fg_run_stats* st = A.stats;
    st->status = FG_OK;
    st->iterations = 0;
    st->reached = A.n;
    st->edges_inspected = 0;
    st->direction_switches = 0;
    st->grid_blocks = 0;
    st->clock_khz = A.clock_khz;
    st->t_start = (int64_t)wall_clock64();
  }
}

__global__ void pr_reset_kernel(PrCtl* c) {
  if (threadIdx.x == 0) {
    PrCtl z;
    memset(&z, 0, sizeof(z));
    *c = z;
  }
}

// Sum of x over the lanes of this lane's run of equal `key` up to this
// lane (runs are adjacent lanes; `start` = the run's first lane), in a
// fixed order.
__device__ __forceinline__ double seg_incl_sum(double x, int lane, int start) {
#pragma unroll
  for (int dd = 1; dd < FG_WAVE; dd <<= 1) {
    const double y = __shfl_up(x, dd, FG_WAVE);
    if (lane - dd >= start) x += y;
  }
  return x;
}

// Sum of cur[col[i]] for i = first, first + stride, ... < end, with four
// independent partial sums so that four gathers per thread are in flight
// (a long row is otherwise a chain of dependent column-then-value loads,
// and the longest row held its workgroup for most of an iteration; eight
// partial sums measured no faster); the order of the additions is fixed.
__device__ __forceinline__ double strided_gather_sum(const double* cur, const int32_t* col,
                                                     uint32_t first, uint32_t end, uint32_t stride) {
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  // unsigned places: a row may end at 2^31 - 1
  uint32_t i = first;
  const uint32_t last = end > 3 * stride ? end - 3 * stride : 0u;
  for (; i < last; i += 4 * stride) {
    const int32_t c0 = col[i];
    const int32_t c1 = col[i + stride];
    const int32_t c2 = col[i + 2 * stride];
    const int32_t c3 = col[i + 3 * stride];
    a0 += cur[c0];
    a1 += cur[c1];
    a2 += cur[c2];
    a3 += cur[c3];
  }
  for (; i < end; i += stride) a0 += cur[col[i]];
  return (a0 + a1) + (a2 + a3);
}

__global__ __launch_bounds__(PR_BT) void pr_iter_kernel(PrArgs A, int32_t it) {
  __shared__ int32_t s_item;
  __shared__ int s_last;
  __shared__ double s_red[PR_BT / FG_WAVE];
  // short rows of each wave's 64 vertices: exclusive prefix of their
  // lengths, their first entries, their sums
  __shared__ int32_t s_sc[PR_BT / FG_WAVE][FG_WAVE];
  __shared__ int32_t s_sb[PR_BT / FG_WAVE][FG_WAVE];
  __shared__ double s_acc[PR_BT / FG_WAVE][FG_WAVE];
  PrCtl* C = A.ctl;
  if (C->done) return;
  const int par = it & 1;
  const double* cur = A.contrib[par];
  double* nxt = A.contrib[par ^ 1];
  const int lane = fg_lane();
  const int wid = threadIdx.x / FG_WAVE;
  const int32_t nlong = C->nlong;
  const int64_t ngroups = ((int64_t)A.n + PR_BT - 1) / PR_BT;
  const int64_t items = (int64_t)nlong + ngroups;
  unsigned long long nc = 0;
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) s_item = (int32_t)atomicAdd(&C->next_item[par], 1u);
    __syncthreads();
    const int64_t item = s_item;
    if (item >= items) break;
    if (item < nlong) {
      // one long row, the whole workgroup
      const int32_t v = A.longrows[item];
      const int32_t b = A.off[v], e = A.off[v + 1];
      double acc = strided_gather_sum(cur, A.col, (uint32_t)b + threadIdx.x, e, PR_BT);
      acc = wave_sum_f64(acc);
      if (lane == 0) s_red[wid] = acc;
      __syncthreads();
      if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < PR_BT / FG_WAVE; ++w) t += s_red[w];
        nc += pr_update(A, nxt, v, e - b, t);
      }
      continue;
    }
    // 256 consecutive vertices, 64 per wave
    const int64_t v64 = (item - nlong) * PR_BT + threadIdx.x;
    const int32_t v = (int32_t)v64;
    int32_t b = 0, deg = 0;
    if (v64 < A.n) {
      b = A.off[v];
      deg = A.off[v + 1] - b;
    }
    {
      // short rows: the wave's rows laid end to end and taken 64 entries
      // per step, one per lane (all the contribution loads of a step in
      // flight together); a step's lanes of one row (adjacent) are summed
      // by a segmented scan and its last lane adds the part to the row's
      // sum, so every row is summed in a fixed order
      const int32_t ds = (v64 < A.n && deg < FG_WAVE) ? deg : 0;
      const int32_t incl = fg_wave_incl_scan(ds);
      const int32_t T = __builtin_amdgcn_readlane(incl, FG_WAVE - 1);
      int32_t* sc = s_sc[wid];
      int32_t* sb = s_sb[wid];
      double* sacc = s_acc[wid];
      sc[lane] = incl - ds;
      sb[lane] = b;
      sacc[lane] = 0.0;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
      for (int32_t t0 = 0; t0 < T; t0 += FG_WAVE) {
        const int32_t t = t0 + lane;
        double x = 0.0;
        int32_t key = -1 - lane;  // lanes past the end: runs of their own
        if (t < T) {
          const int32_t j = fgk::upper_idx(sc, FG_WAVE, t);
          // t - sc[j] < the length of row j: the entry lies inside its row
          x = cur[A.col[sb[j] + (t - sc[j])]];
          key = j;
        }
        const int32_t kp = __shfl_up(key, 1, FG_WAVE);
        const int32_t kn = __shfl_down(key, 1, FG_WAVE);
        const bool head = lane == 0 || kp != key;
        const bool tail = lane == FG_WAVE - 1 || kn != key;
        const uint64_t H = __ballot(head);
        const uint64_t upto = lane == FG_WAVE - 1 ? ~0ull : ((2ull << lane) - 1ull);
        const int start = 63 - __builtin_clzll(H & upto);
        x = seg_incl_sum(x, lane, start);
        if (tail && key >= 0) sacc[key] += x;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
      if (v64 < A.n && deg < FG_WAVE) nc += pr_update(A, nxt, v, deg, sacc[lane]);
    }
    // medium rows: one at a time, the whole wave across the row
    uint64_t med = __ballot(deg >= FG_WAVE && deg < PR_LONG);
    while (med) {
      const int l = __builtin_ctzll(med);
      med &= med - 1;
      const int32_t ub = __shfl(b, l, FG_WAVE);
      const int32_t ud = __shfl(deg, l, FG_WAVE);
      double acc = 0.0;
      acc = strided_gather_sum(cur, A.col, (uint32_t)ub + lane, ub + ud, FG_WAVE);
      acc = wave_sum_f64(acc);
      if (lane == l) nc += pr_update(A, nxt, v, ud, acc);
    }
  }
  nc = fg_wave_sum(nc);
  if (lane == 0 && nc) atomicAdd(&C->notconv[par], nc);

  // the last workgroup closes the iteration
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  if (threadIdx.x == 0) s_last = atomicAdd(&C->blocks_done, 1u) == gridDim.x - 1;
  __syncthreads();
  if (!s_last || threadIdx.x != 0) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  const unsigned long long above =
      __hip_atomic_load(&C->notconv[par], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (A.stats) {
    fg_run_stats* st = A.stats;
    if (it < FG_TRACE_MAX) {
      st->dir[it] = 0;
      st->frontier[it] = (int64_t)above;
      st->inspected[it] = A.m;
      st->t_end[it] = (int64_t)wall_clock64();
    }
    st->iterations = it + 1;
    st->edges_inspected += A.m;
  }
  C->iterations = it + 1;
  if (A.tol > 0.0 && above == 0) C->done = 1;
  C->notconv[par ^ 1] = 0;
  C->next_item[par] = 0;
  C->blocks_done = 0;
}

// ------------------------------------------------------- the planned form

constexpr int PP_BT = 1024;
constexpr int PP_WAVES = PP_BT / FG_WAVE;
constexpr int PP_XCD = 8;       // column classes, one per XCD
constexpr int PP_HOT = 18432;   // contributions in LDS (144 KB: one workgroup per CU)
constexpr int PP_SHORT = 64;    // shorter rows: one lane each, 64 rows per slice
constexpr int PP_SEG = 2048;    // rows of at least this many entries are cut into segments
constexpr int PP_OCT = 8;       // degree classes per power of two from PP_SHORT on
constexpr int PP_LONGB = (31 - 6) * PP_OCT;      // classes of degrees >= 64
constexpr int PP_BUCKETS = PP_LONGB + PP_SHORT;  // then one for 63, 62, ..., 0
constexpr int PP_PER = 4;       // vertices per thread of the numbering passes
constexpr int PP_TILE = PP_BT * PP_PER;
constexpr int PP_PAD = PP_SHORT * FG_WAVE;  // most entries that pad the slices
// On large graphs the plan costs 1.5 iterations of the direct form and each
// iteration saves two thirds of one: two iterations 2604 us direct and 2704
// planned, three 3877 and 3119 (R-MAT 22), 573 and 584, 858 and 729 (uniform
// random, 16.8 M entries).  On small ones an iteration's work counter costs
// more than the plan: 9 M entries 587 and 231, 0.5 M 253 and 120.
constexpr int PP_MIN_ITER = 3;
constexpr int64_t PP_SMALL_M = 10 << 20;

struct PrPlan {
  uint32_t count[PP_BUCKETS];   // vertices per class, then the class's first number
  uint32_t rows_seg;            // rows [0, rows_seg) have at least PP_SEG entries,
  uint32_t rows_1024;           // up to here 1024,
  uint32_t rows_256;            // 256,
  uint32_t rows_long;           // PP_SHORT;
  uint32_t rows;                // up to here at least one; the rest are empty
  uint32_t next_entry;          // allocation of the long rows' entries
  uint32_t next_seg;            // ... and of the segments of rows [0, rows_seg)
  uint32_t slice_first[PP_SHORT];  // first slice whose first row has this degree
  uint32_t slice_base[PP_SHORT];   // its entries' place
  unsigned long long closed;    // workgroups done << 40 | vertices above the threshold
  int32_t done;
};

struct PrPlanned {
  PrPlan* plan;
  uint32_t tiles, classlen, segcap;  // classlen: contributions per column class
  uint32_t* hist;    // [class of degree][tile]
  double* rk;        // rank by new number
  double* contrib[2];  // [column class][number / 8]; 0 from number `rows` on
  int32_t* newid;    // vertex -> new number
  int32_t* deg;      // by new number
  int32_t* beg;      // first entry in the graph's columns
  uint32_t* place;   // long rows: first entry in `ncol`
  uint32_t* seg0;    // rows [0, rows_seg): first segment
  uint2* sub;        // [column class][segment]: first entry in `ncol`, entries
  double* part;      // [column class][segment]: partial sums
  uint32_t* slice;   // slices: first entry in `ncol`
  int32_t* ncol;     // renumbered columns
  uint32_t* bar;     // grid barrier of pp_loop_kernel
};

// Classes in falling order of degree: eight per power of two from 64 on,
// then 63 down to 0 each by itself.
__device__ __forceinline__ int pp_bucket(int32_t d) {
  if (d < PP_SHORT) return PP_BUCKETS - 1 - d;
  const int lg = 31 - __builtin_clz(d);
  return PP_LONGB - 1 - ((lg - 6) * PP_OCT + ((d >> (lg - 3)) & (PP_OCT - 1)));
}

// Where the contribution of number x lies.
__device__ __forceinline__ uint32_t pp_slot(uint32_t x, uint32_t classlen) {
  return (x & (PP_XCD - 1)) * classlen + x / PP_XCD;
}

__global__ __launch_bounds__(PP_BT) void pp_clear_kernel(PrArgs A, PrPlan* P, uint32_t* bar) {
  uint32_t* w = (uint32_t*)P;
  for (uint32_t i = threadIdx.x; i < sizeof(PrPlan) / 4; i += PP_BT) w[i] = 0;
  if (bar)
    for (uint32_t i = threadIdx.x; i < FG_BAR_WORDS; i += PP_BT) bar[i] = 0;
  if (threadIdx.x == 0 && A.stats) {
    fg_run_stats* st = A.stats;
    st->status = FG_OK;
    st->iterations = 0;
    st->reached = A.n;
    st->edges_inspected = 0;
    st->direction_switches = 0;
    st->grid_blocks = 0;
    st->clock_khz = A.clock_khz;
    st->t_start = (int64_t)wall_clock64();
  }
}

// The numbering is a stable counting sort by class (a vertex's number, and
// with it the column class that an entry falls into, does not change from
// call to call): counts per tile, their prefix per class, the classes'
// places, ranks within the tile.
__global__ __launch_bounds__(PP_BT) void pp_count_kernel(int32_t n, const int32_t* __restrict__ off,
                                                         PrPlanned Q) {
  __shared__ uint32_t s_cnt[PP_BUCKETS];
  for (int i = threadIdx.x; i < PP_BUCKETS; i += PP_BT) s_cnt[i] = 0;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < PP_PER; ++r) {
    const int64_t v = (int64_t)blockIdx.x * PP_TILE + r * PP_BT + threadIdx.x;
    if (v < n) atomicAdd(&s_cnt[pp_bucket(off[v + 1] - off[v])], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < PP_BUCKETS; i += PP_BT)
    Q.hist[(size_t)i * Q.tiles + blockIdx.x] = s_cnt[i];
}

__global__ __launch_bounds__(PP_BT) void pp_prefix_kernel(PrPlanned Q) {
  __shared__ uint32_t s_red[PP_WAVES + 1];
  uint32_t* h = Q.hist + (size_t)blockIdx.x * Q.tiles;
  uint32_t carry = 0;
  for (uint32_t t0 = 0; t0 < Q.tiles; t0 += PP_BT) {
    const uint32_t t = t0 + threadIdx.x;
    const uint32_t c = t < Q.tiles ? h[t] : 0u;
    uint32_t all = 0;
    const uint32_t ex = fg_block_excl_scan<PP_BT>(c, s_red, &all);
    if (t < Q.tiles) h[t] = carry + ex;
    carry += all;
  }
  if (threadIdx.x == 0) Q.plan->count[blockIdx.x] = carry;
}

// Places of the classes and of the slices (one workgroup).
constexpr int PP_SCAN_BT = 512;
static_assert(PP_BUCKETS < PP_SCAN_BT, "one thread per class");
__global__ __launch_bounds__(PP_SCAN_BT) void pp_scan_kernel(int64_t m, PrPlan* __restrict__ P) {
  __shared__ uint32_t s[PP_SCAN_BT];
  __shared__ unsigned long long s_red64[PP_SCAN_BT / FG_WAVE + 1];
  __shared__ uint32_t s_red[PP_SCAN_BT / FG_WAVE + 1];
  const int b = threadIdx.x;
  const uint32_t c = b < PP_BUCKETS ? P->count[b] : 0u;
  uint32_t all = 0;
  s[b] = fg_block_excl_scan<PP_SCAN_BT>(c, s_red, &all);
  const unsigned long long shorts = fg_block_sum<PP_SCAN_BT>(
      b >= PP_LONGB && b < PP_BUCKETS ? (unsigned long long)c * (PP_BUCKETS - 1 - b) : 0ull, s_red64);
  __syncthreads();
  if (b < PP_BUCKETS) P->count[b] = s[b];
  if (b == 0) {
    P->rows_seg = s[PP_LONGB - (11 - 6) * PP_OCT];
    P->rows_1024 = s[PP_LONGB - (10 - 6) * PP_OCT];
    P->rows_256 = s[PP_LONGB - (8 - 6) * PP_OCT];
    P->rows_long = s[PP_LONGB];
    P->rows = s[PP_BUCKETS - 1];
  }
  // slices: 64 consecutive rows from rows_long on, as wide as their first;
  // thread b looks at degree 63 - b
  const int d = PP_SHORT - 1 - b;
  uint32_t f = 0, l = 0;
  if (d > 0) {
    const uint32_t r0 = s[PP_LONGB];
    f = (s[PP_LONGB + b] - r0 + FG_WAVE - 1) / FG_WAVE;
    l = (s[PP_LONGB + b + 1] - r0 + FG_WAVE - 1) / FG_WAVE;
  }
  const uint32_t base =
      fg_block_excl_scan<PP_SCAN_BT>(d > 0 ? (l - f) * (uint32_t)(d * FG_WAVE) : 0u, s_red, &all);
  if (d > 0) {
    P->slice_first[d] = f;
    P->slice_base[d] = (uint32_t)(m - (int64_t)shorts) + base;
  }
}

__global__ __launch_bounds__(PP_BT) void pp_number_kernel(int32_t n,
                                                          const int32_t* __restrict__ off,
                                                          PrPlanned Q, double inv_n) {
  __shared__ uint32_t s_wc[PP_WAVES][PP_BUCKETS + 1];
  __shared__ uint32_t s_base[PP_BUCKETS + 1];
  __shared__ uint32_t s_entries, s_segs;
  PrPlan* P = Q.plan;
  const int wid = threadIdx.x / FG_WAVE;
  for (int i = threadIdx.x; i <= PP_BUCKETS; i += PP_BT) {
    s_base[i] = i < PP_BUCKETS ? P->count[i] + Q.hist[(size_t)i * Q.tiles + blockIdx.x] : 0u;
    for (int w = 0; w < PP_WAVES; ++w) s_wc[w][i] = 0;
  }
  if (threadIdx.x == 0) s_entries = s_segs = 0;
  __syncthreads();
  int32_t b[PP_PER], d[PP_PER];
  uint32_t at[PP_PER], entry[PP_PER], seg[PP_PER];
#pragma unroll
  for (int r = 0; r < PP_PER; ++r) {
    const int64_t v = (int64_t)blockIdx.x * PP_TILE + r * PP_BT + threadIdx.x;
    d[r] = -1;
    if (v < n) {
      b[r] = off[v];
      d[r] = off[v + 1] - b[r];
    }
    const int k = d[r] < 0 ? PP_BUCKETS : pp_bucket(d[r]);
    uint64_t peers = ~0ull;  // lanes of this wave with the same class
#pragma unroll
    for (int bit = 0; bit < 9; ++bit) {
      const uint64_t m = __ballot((k >> bit) & 1);
      peers &= ((k >> bit) & 1) ? m : ~m;
    }
    const int rank = fg_mbcnt(peers);
    if (rank == 0) s_wc[wid][k] = __popcll(peers);
    __syncthreads();
    for (int i = threadIdx.x; i < PP_BUCKETS; i += PP_BT) {
      uint32_t run = s_base[i];
      for (int w = 0; w < PP_WAVES; ++w) {
        const uint32_t c = s_wc[w][i];
        s_wc[w][i] = run;
        run += c;
      }
      s_base[i] = run;
    }
    __syncthreads();
    at[r] = s_wc[wid][k] + rank;
    if (d[r] >= PP_SHORT) entry[r] = atomicAdd(&s_entries, (uint32_t)d[r]);
    if (d[r] >= PP_SEG) seg[r] = atomicAdd(&s_segs, (uint32_t)fgk::fg_pieces(d[r], PP_SEG));
    __syncthreads();
    for (int i = threadIdx.x; i < PP_BUCKETS; i += PP_BT)
      for (int w = 0; w < PP_WAVES; ++w) s_wc[w][i] = 0;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (s_entries) s_entries = atomicAdd(&P->next_entry, s_entries);
    if (s_segs) s_segs = atomicAdd(&P->next_seg, s_segs);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < PP_PER; ++r) {
    if (d[r] < 0) continue;
    const int64_t v = (int64_t)blockIdx.x * PP_TILE + r * PP_BT + threadIdx.x;
    const uint32_t x = at[r];
    const uint32_t slot = pp_slot(x, Q.classlen);
    Q.newid[v] = (int32_t)x;
    Q.contrib[0][slot] = d[r] > 0 ? inv_n / (double)d[r] : 0.0;
    if (d[r] == 0) {
      Q.contrib[1][slot] = 0.0;
      continue;
    }
    Q.rk[x] = inv_n;
    Q.deg[x] = d[r];
    Q.beg[x] = b[r];
    if (d[r] >= PP_SHORT) Q.place[x] = s_entries + entry[r];
    if (d[r] >= PP_SEG) Q.seg0[x] = s_segs + seg[r];
  }
  // the numbers behind the last vertex
  if (blockIdx.x == 0)
    for (uint32_t x = (uint32_t)n + threadIdx.x; x < Q.classlen * PP_XCD; x += PP_BT)
      Q.contrib[0][pp_slot(x, Q.classlen)] = Q.contrib[1][pp_slot(x, Q.classlen)] = 0.0;
}

// The lanes whose column class is `cls`, from the ballots of its three bits.
__device__ __forceinline__ uint64_t pp_class_mask(int cls, uint64_t valid, uint64_t b0, uint64_t b1,
                                                  uint64_t b2) {
  return valid & ((cls & 1) ? b0 : ~b0) & ((cls & 2) ? b1 : ~b1) & ((cls & 4) ? b2 : ~b2);
}

// One segment (up to PP_SEG entries) by a wave: its columns' new numbers into
// LDS while each class is counted, then out class by class, every class in
// CSR order and without the three bits that are the same throughout it.
__device__ __forceinline__ void pp_segment(const PrPlanned& Q, const int32_t* c, uint32_t place,
                                           int32_t len, uint32_t s, int32_t* tmp, uint32_t* run) {
  const int lane = fg_lane();
  uint32_t cnt = 0;  // lane j < 8: entries of class j
  for (int32_t k0 = 0; k0 < len; k0 += 4 * FG_WAVE) {
    int32_t i[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int32_t k = k0 + r * FG_WAVE + lane;
      i[r] = k < len ? __builtin_nontemporal_load(c + k) : 0;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) i[r] = Q.newid[i[r]];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int32_t k = k0 + r * FG_WAVE + lane;
      if (k < len) tmp[k] = i[r];
      cnt += __popcll(pp_class_mask(lane, __ballot(k < len), __ballot(i[r] & 1),
                                    __ballot(i[r] & 2), __ballot(i[r] & 4)));
    }
  }
  const int32_t mine = lane < PP_XCD ? (int32_t)cnt : 0;
  const uint32_t first = (uint32_t)(fg_wave_incl_scan(mine) - mine);
  if (lane < PP_XCD) {
    Q.sub[(size_t)lane * Q.segcap + s] = make_uint2(place + first, cnt);
    run[lane] = first;
  }
  fgk::wave_lds_fence();
  int32_t* o = Q.ncol + place;
  for (int32_t k0 = 0; k0 < len; k0 += FG_WAVE) {
    const bool in = k0 + lane < len;
    const int32_t x = in ? tmp[k0 + lane] : 0;
    const uint64_t v = __ballot(in), b0 = __ballot(x & 1), b1 = __ballot(x & 2),
                   b2 = __ballot(x & 4);
    const int cls = x & (PP_XCD - 1);
    if (in) o[run[cls] + fg_mbcnt(pp_class_mask(cls, v, b0, b1, b2))] = x / PP_XCD;
    fgk::wave_lds_fence();
    if (lane < PP_XCD) run[lane] += __popcll(pp_class_mask(lane, v, b0, b1, b2));
    fgk::wave_lds_fence();
  }
}

// The columns under their new numbers: long rows by segment and class,
// slices entry by entry across their 64 rows (entries past a row's end read
// the contribution 0 of the first number behind the rows).
__global__ __launch_bounds__(PP_BT) void pp_columns_kernel(const int32_t* __restrict__ col,
                                                           PrPlanned Q) {
  __shared__ int32_t s_tmp[PP_WAVES][PP_SEG];
  __shared__ uint32_t s_run[PP_WAVES][PP_XCD];
  const PrPlan* P = Q.plan;
  const int lane = fg_lane();
  const int wid = threadIdx.x / FG_WAVE;
  const uint32_t gw = wid * gridDim.x + blockIdx.x;
  const uint32_t W = gridDim.x * PP_WAVES;
  const uint32_t rs = P->rows_seg, rl = P->rows_long, rows = P->rows, segs = P->next_seg;
  for (uint32_t x = blockIdx.x; x < rs; x += gridDim.x) {
    const int32_t d = Q.deg[x];
    const int32_t pieces = fgk::fg_pieces(d, PP_SEG);
    for (int32_t j = wid; j < pieces; j += PP_WAVES) {
      const int32_t at = j * PP_SEG;
      pp_segment(Q, col + Q.beg[x] + at, Q.place[x] + at, d - at < PP_SEG ? d - at : PP_SEG,
                 Q.seg0[x] + j, s_tmp[wid], s_run[wid]);
    }
  }
  for (uint32_t x = rs + gw; x < rl; x += W)
    pp_segment(Q, col + Q.beg[x], Q.place[x], Q.deg[x], segs + (x - rs), s_tmp[wid], s_run[wid]);
  for (uint32_t s = gw; (uint64_t)s * FG_WAVE < rows - rl; s += W) {
    const uint32_t x = rl + s * FG_WAVE + lane;
    const int32_t d = x < rows ? Q.deg[x] : 0;
    const int32_t* c = col + (x < rows ? Q.beg[x] : 0);
    const int32_t w = __builtin_amdgcn_readfirstlane(d);
    const uint32_t base = P->slice_base[w] + (s - P->slice_first[w]) * (uint32_t)(w * FG_WAVE);
    if (lane == 0) Q.slice[s] = base;
    int32_t* o = Q.ncol + base + lane;
    for (int32_t k0 = 0; k0 < w; k0 += 8) {
      int32_t i[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) i[r] = k0 + r < d ? c[k0 + r] : 0;
#pragma unroll
      for (int r = 0; r < 8; ++r) i[r] = k0 + r < d ? Q.newid[i[r]] : (int32_t)rows;
#pragma unroll
      for (int r = 0; r < 8; ++r)
        if (k0 + r < w) __builtin_nontemporal_store(i[r], o + (k0 + r) * FG_WAVE);
    }
  }
}

// A contribution: the first `nhot` are in LDS, the others are gathered.  The
// lanes that find theirs in LDS all read a contribution 0 behind the last
// row instead of a line of their own, so the gather costs what the other
// lanes cost and there is no branch between the loads of a step.
struct PpClassCur {  // by number / 8 within a column class
  const double* cur;
  const double* hot;  // LDS
  uint32_t nhot, zero;
  __device__ __forceinline__ double operator[](uint32_t i) const {
    const bool h = i < nhot;
    const double g = cur[h ? zero : i];
    const double l = hot[h ? i : 0u];
    return h ? l : g;
  }
};

struct PpCur {  // by number
  const double* cur;
  const double* hot;  // LDS
  uint32_t nhot, zero, classlen;
  __device__ __forceinline__ double operator[](uint32_t i) const {
    const bool h = i < nhot;
    const double g = cur[pp_slot(h ? zero : i, classlen)];
    const double l = hot[h ? i : 0u];
    return h ? l : g;
  }
};

// The columns are read past the caches, which are left to the contributions.
__device__ __forceinline__ uint32_t pp_col(const int32_t* p) {
  return (uint32_t)__builtin_nontemporal_load(p);
}

// The sums of segments [lo, hi) of a column class: G lanes per segment, 64/G
// segments per unit, the wave's units gw, gw + W, ... in batches of N.  A
// unit is a chain of dependent loads (its place, its columns, their
// contributions: 2.5 us) with hardly more than one load of each kind, and a
// CU holds only 16 waves beside the LDS table, so N units are taken together
// and the next places are on their way meanwhile.  U columns per lane cover
// most segments; the loop behind takes what is longer.
template <int G, int U, int N>
__device__ __forceinline__ void pp_segment_sums(const PrPlanned& Q, const PpClassCur& cur,
                                                const uint2* sub, double* part, uint32_t lo,
                                                uint32_t hi, uint32_t gw, uint32_t W) {
  constexpr uint32_t PER = FG_WAVE / G;
  const int lane = fg_lane();
  const uint32_t units = (hi - lo + PER - 1) / PER;
  if (gw >= units) return;
  const uint32_t l0 = lane & (G - 1);
  uint2 r[N];
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const uint32_t s = lo + (gw + q * W) * PER + lane / G;
    r[q] = s < hi ? sub[s] : make_uint2(0, 0);
  }
  for (uint32_t u = gw; u < units; u += N * W) {
    uint32_t i[N][U];
    double y[N][U], acc[N];
    uint2 now[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
      now[q] = r[q];
#pragma unroll
      for (int k = 0; k < U; ++k)
        i[q][k] = l0 + k * G < now[q].y ? pp_col(Q.ncol + now[q].x + l0 + k * G) : cur.zero;
      const uint32_t s = lo + (u + (N + q) * W) * PER + lane / G;
      r[q] = s < hi ? sub[s] : make_uint2(0, 0);
    }
#pragma unroll
    for (int q = 0; q < N; ++q)
#pragma unroll
      for (int k = 0; k < U; ++k) y[q][k] = cur[i[q][k]];
#pragma unroll
    for (int q = 0; q < N; ++q) {
#pragma unroll
      for (int w = U / 2; w > 0; w >>= 1)
#pragma unroll
        for (int k = 0; k < w; ++k) y[q][k] += y[q][k + w];
      acc[q] = y[q][0];
      for (uint32_t k = l0 + U * G; k < now[q].y; k += G) acc[q] += cur[pp_col(Q.ncol + now[q].x + k)];
    }
#pragma unroll
    for (int d = G / 2; d > 0; d >>= 1)
#pragma unroll
      for (int q = 0; q < N; ++q) acc[q] += __shfl_xor(acc[q], d, FG_WAVE);
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const uint32_t s = lo + (u + q * W) * PER + lane / G;
      if (l0 == 0 && s < hi) part[s] = acc[q];
    }
  }
}

// The long rows' partial sums.  Workgroup b takes the entries of column
// class b mod 8 of every segment: consecutive workgroups lie on different
// XCDs, so each XCD's L2 (4 MB) has to hold an eighth of the contributions
// and the LDS of its CUs the first 18 k of that eighth, over 140 k numbers
// in all, which nine tenths of an R-MAT graph's entries ask for.  (Which XCD
// a workgroup is on matters for speed alone.)  Segments are dealt round in
// falling order of their rows' length.
__device__ __forceinline__ void pp_long(const PrPlanned& Q, int32_t it, double* s_hot) {
  const PrPlan* P = Q.plan;
  const uint32_t rs = P->rows_seg, segs = P->next_seg;
  const uint32_t s1 = segs + (P->rows_1024 - rs), s2 = segs + (P->rows_256 - rs);
  const uint32_t s3 = segs + (P->rows_long - rs);
  if (s3 == 0) return;
  const uint32_t cls = blockIdx.x & (PP_XCD - 1);
  const uint32_t bi = blockIdx.x / PP_XCD, nb = gridDim.x / PP_XCD;
  PpClassCur cur{Q.contrib[it & 1] + (size_t)cls * Q.classlen, s_hot,
                 Q.classlen < (uint32_t)PP_HOT ? Q.classlen : (uint32_t)PP_HOT, Q.classlen - 1};
  for (uint32_t i = threadIdx.x; i < cur.nhot; i += PP_BT) s_hot[i] = cur.cur[i];
  __syncthreads();
  const uint2* sub = Q.sub + (size_t)cls * Q.segcap;
  double* part = Q.part + (size_t)cls * Q.segcap;
  const uint32_t W = nb * PP_WAVES, gw = (threadIdx.x / FG_WAVE) * nb + bi;
  pp_segment_sums<64, 4, 4>(Q, cur, sub, part, 0, s1, gw, W);
  pp_segment_sums<16, 8, 2>(Q, cur, sub, part, s1, s2, gw, W);
  pp_segment_sums<8, 4, 4>(Q, cur, sub, part, s2, s3, gw, W);
}

__global__ __launch_bounds__(PP_BT) void pp_long_kernel(PrPlanned Q, int32_t it) {
  __shared__ double s_hot[PP_HOT];
  if (Q.plan->done) return;
  pp_long(Q, it, s_hot);
}

// The update of row x from its accumulated sum, as pr_update.
__device__ __forceinline__ uint32_t pp_update(const PrArgs& A, const PrPlanned& Q, double* nxt,
                                              uint32_t x, double acc) {
  const double nr = __dadd_rn(A.base, __dmul_rn(A.d, acc));
  const double old = Q.rk[x];
  const double diff = nr > old ? __dsub_rn(nr, old) : __dsub_rn(old, nr);
  Q.rk[x] = nr;
  nxt[pp_slot(x, Q.classlen)] = nr / (double)Q.deg[x];
  return diff > __dmul_rn(A.tol, old) ? 1u : 0u;
}

// The rest of an iteration: the slices (a lane per row, the first 18 k
// contributions of all classes in LDS), the long rows' partial sums taken
// together, every row's update, and the close of the iteration.  All are
// dealt round over the waves, so there is no work counter (one atomic per
// 256 vertices on one address was 190 us of the direct form's iteration on
// R-MAT 22).
__device__ __forceinline__ void pp_iter(const PrArgs& A, const PrPlanned& Q, int32_t it,
                                        double* s_hot, uint32_t* s_nc) {
  PrPlan* P = Q.plan;
  double* nxt = Q.contrib[(it & 1) ^ 1];
  const int lane = fg_lane();
  const int wid = threadIdx.x / FG_WAVE;
  const uint32_t gw = wid * gridDim.x + blockIdx.x;  // consecutive waves: other workgroups
  const uint32_t W = gridDim.x * PP_WAVES;
  const uint32_t rs = P->rows_seg, rl = P->rows_long, rows = P->rows, segs = P->next_seg;
  PpCur cur{Q.contrib[it & 1], s_hot, rows < (uint32_t)PP_HOT ? rows : (uint32_t)PP_HOT, rows,
            Q.classlen};
  if (rl < rows)
    for (uint32_t i = threadIdx.x; i < cur.nhot; i += PP_BT)
      s_hot[i] = cur.cur[pp_slot(i, Q.classlen)];
  __syncthreads();
  const uint32_t u1 = rs + (rl - rs + FG_WAVE - 1) / FG_WAVE;
  const uint32_t u2 = u1 + (rows - rl + FG_WAVE - 1) / FG_WAVE;
  uint32_t nc = 0;
  for (uint32_t u = gw; u < u2; u += W) {
    if (u < rs) {
      // a row of several segments, a wave across its partial sums
      const uint32_t k = (uint32_t)fgk::fg_pieces(Q.deg[u], PP_SEG) * PP_XCD;
      const double* p = Q.part + Q.seg0[u];
      double acc = 0.0;
      for (uint32_t i = lane; i < k; i += FG_WAVE)
        acc += p[(size_t)(i & (PP_XCD - 1)) * Q.segcap + i / PP_XCD];
      acc = wave_sum_f64(acc);
      if (lane == 0) nc += pp_update(A, Q, nxt, u, acc);
    } else if (u < u1) {
      const uint32_t x = rs + (u - rs) * FG_WAVE + lane;
      if (x < rl) {
        const double* p = Q.part + segs + (x - rs);
        double y[PP_XCD];
#pragma unroll
        for (int k = 0; k < PP_XCD; ++k) y[k] = p[(size_t)k * Q.segcap];
        nc += pp_update(A, Q, nxt, x,
                        ((y[0] + y[1]) + (y[2] + y[3])) + ((y[4] + y[5]) + (y[6] + y[7])));
      }
    } else {
      const uint32_t x = rl + (u - u1) * FG_WAVE + lane;
      const int32_t w = __builtin_amdgcn_readfirstlane(Q.deg[x < rows ? x : rl]);
      const int32_t* c = Q.ncol + Q.slice[u - u1] + lane;
      double acc = 0.0;
      int32_t k = 0;
      for (; k + 8 <= w; k += 8) {
        uint32_t i[8];
        double y[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) i[r] = pp_col(c + (k + r) * FG_WAVE);
#pragma unroll
        for (int r = 0; r < 8; ++r) y[r] = cur[i[r]];
        acc += ((y[0] + y[1]) + (y[2] + y[3])) + ((y[4] + y[5]) + (y[6] + y[7]));
      }
      if (k < w) {
        uint32_t i[8];
        double y[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) i[r] = k + r < w ? pp_col(c + (k + r) * FG_WAVE) : cur.zero;
#pragma unroll
        for (int r = 0; r < 8; ++r) y[r] = cur[i[r]];
        acc += ((y[0] + y[1]) + (y[2] + y[3])) + ((y[4] + y[5]) + (y[6] + y[7]));
      }
      if (x < rows) nc += pp_update(A, Q, nxt, x, acc);
    }
  }
  nc = (uint32_t)fg_wave_sum((int32_t)nc);
  if (lane == 0) s_nc[wid] = nc;
  __syncthreads();
  if (threadIdx.x != 0) return;
  unsigned long long mine = 0;
  for (int w = 0; w < PP_WAVES; ++w) mine += s_nc[w];
  // one atomic carries the arrival and the count; the last workgroup closes
  // the iteration
  const unsigned long long old = atomicAdd(&P->closed, (1ull << 40) | mine);
  if ((old >> 40) != gridDim.x - 1) return;
  unsigned long long above = (old & ((1ull << 40) - 1)) + mine;
  if (it == 0) {
    // the vertices without edges go from 1/n to (1 - d)/n here and stay there
    const double first = 1.0 / (double)A.n;
    const double diff = A.base > first ? __dsub_rn(A.base, first) : __dsub_rn(first, A.base);
    if (diff > __dmul_rn(A.tol, first)) above += (uint32_t)A.n - rows;
  }
  if (A.stats) {
    fg_run_stats* st = A.stats;
    if (it < FG_TRACE_MAX) {
      st->dir[it] = 0;
      st->frontier[it] = (int64_t)above;
      st->inspected[it] = A.m;
      st->t_end[it] = (int64_t)wall_clock64();
    }
    st->iterations = it + 1;
    st->edges_inspected += A.m;
  }
  if (A.tol > 0.0 && above == 0)
    __hip_atomic_store(&P->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(&P->closed, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(PP_BT) void pp_iter_kernel(PrArgs A, PrPlanned Q, int32_t it) {
  __shared__ double s_hot[PP_HOT];
  __shared__ uint32_t s_nc[PP_WAVES];
  if (Q.plan->done) return;
  pp_iter(A, Q, it, s_hot, s_nc);
}

// All iterations in one co-resident launch, for runs that may stop early: the
// launches left after the stop cost 3.4 us each, and the planned form has two
// per iteration (at most 1000 iterations, stopped after 7: 7.0 ms on 20 k
// vertices, 3.3 with the direct form's one).  An iteration takes 5 to 30 us
// longer for its barriers, with which at most 100 iterations break even after
// about ten: 300 k vertices, 3, 7 and 18 of them 370, 633 and 1350 us, as
// launches 618, 720 and 1125.  (Stores past the L2 in place of its write-back
// at the barriers: 2 to 12 % less up to 20 k vertices, 4 to 48 % more above.)
__global__ __launch_bounds__(PP_BT) void pp_loop_kernel(PrArgs A, PrPlanned Q, int32_t max_iter,
                                                        int32_t longs) {
  __shared__ double s_hot[PP_HOT];
  __shared__ uint32_t s_nc[PP_WAVES];
  __shared__ int s_flag;
  fg_grid_sync gs{Q.bar, gridDim.x, 0u};
  bool ok = true;
  for (int32_t it = 0; it < max_iter && ok; ++it) {
    if (longs) {
      pp_long(Q, it, s_hot);
      if (!(ok = gs.sync(&s_flag))) break;
    }
    pp_iter(A, Q, it, s_hot, s_nc);
    if (!(ok = gs.sync(&s_flag))) break;
    if (__hip_atomic_load(&Q.plan->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
  }
  if (!ok && blockIdx.x == 0 && threadIdx.x == 0 && A.stats) A.stats->status = FG_EDEVICE;
}

__global__ __launch_bounds__(PP_BT) void pp_ranks_kernel(PrArgs A, PrPlanned Q) {
  const uint32_t rows = Q.plan->rows;
  for (int64_t v = (int64_t)blockIdx.x * PP_BT + threadIdx.x; v < A.n;
       v += (int64_t)gridDim.x * PP_BT) {
    const uint32_t x = (uint32_t)Q.newid[v];
    A.rank[v] = x < rows ? Q.rk[x] : A.base;
  }
}

struct PrLayout {
  double* contrib0;
  double* contrib1;
  int32_t* longrows;
  PrCtl* ctl;
  size_t bytes;
};

PrLayout pr_layout(const fg_graph* g, void* ws) {
  fg_carver c(ws);
  PrLayout L;
  L.contrib0 = c.take<double>(g->n);
  L.contrib1 = c.take<double>(g->n);
  L.longrows = c.take<int32_t>(g->n);
  L.ctl = c.take<PrCtl>(1);
  L.bytes = c.used;
  return L;
}

// The planned form's workspace (it does not share the direct form's); *loop:
// with the barrier of the one-launch loop behind it.
size_t pr_planned_layout(const fg_graph* g, void* ws, PrPlanned* Q, size_t* loop) {
  fg_carver c(ws);
  const size_t n = (size_t)g->n, m = (size_t)g->m;
  Q->tiles = (uint32_t)((n + PP_TILE - 1) / PP_TILE);
  Q->classlen = (uint32_t)(n / PP_XCD + 2);  // the last number of each class is behind n
  // rows of 64 entries and more, and the segments of those of PP_SEG and more
  Q->segcap = (uint32_t)(m / PP_SHORT + 2 * (m / PP_SEG) + 2);
  Q->plan = c.take<PrPlan>(1);
  Q->hist = c.take<uint32_t>((size_t)PP_BUCKETS * Q->tiles);
  Q->rk = c.take<double>(n);
  Q->contrib[0] = c.take<double>((size_t)Q->classlen * PP_XCD);
  Q->contrib[1] = c.take<double>((size_t)Q->classlen * PP_XCD);
  Q->newid = c.take<int32_t>(n);
  Q->deg = c.take<int32_t>(n);
  Q->beg = c.take<int32_t>(n);
  Q->place = c.take<uint32_t>(m / PP_SHORT + 1);
  Q->seg0 = c.take<uint32_t>(m / PP_SEG + 1);
  Q->sub = c.take<uint2>((size_t)Q->segcap * PP_XCD);
  Q->part = c.take<double>((size_t)Q->segcap * PP_XCD);
  Q->slice = c.take<uint32_t>(n / FG_WAVE + 1);
  Q->ncol = c.take<int32_t>(m + PP_PAD);
  const size_t bytes = c.used;
  Q->bar = c.take<uint32_t>(FG_BAR_WORDS);
  *loop = c.used;
  return bytes;
}

}  // namespace

size_t fg_pr_workspace_bytes(const fg_graph* g) {
  PrPlanned Q;
  size_t loop;
  pr_planned_layout(g, nullptr, &Q, &loop);
  const size_t direct = pr_layout(g, nullptr).bytes;
  return loop > direct ? loop : direct;
}

extern "C" fg_status fg_pagerank(const fg_graph* g, double damping, double tol, int32_t max_iter,
                                 void* ws, size_t ws_bytes, double* rank, fg_run_stats* stats,
                                 void* stream) {
  if (!g || !rank || !ws) return fg_set_error(FG_EINVAL, "fg_pagerank: NULL argument");
  if (!g->symmetric)
    return fg_set_error(FG_EUNSUPPORTED, "fg_pagerank: needs an undirected graph (FG_SYMMETRIC)");
  if (!(damping >= 0.0 && damping <= 1.0))
    return fg_set_error(FG_EINVAL, "fg_pagerank: damping %g outside [0, 1]", damping);
  if (!(tol >= 0.0)) return fg_set_error(FG_EINVAL, "fg_pagerank: tol %g < 0", tol);
  if (max_iter < 0 || max_iter > 100000)
    return fg_set_error(FG_EINVAL, "fg_pagerank: max_iter %d outside [0, 100000]", max_iter);
  PrLayout L = pr_layout(g, ws);
  FG_CHECK_WS_ALIGN(ws, "fg_pagerank");
  if (ws_bytes < L.bytes)
    return fg_set_error(FG_ENOMEM, "fg_pagerank: workspace of %zu bytes < required %zu",
                        ws_bytes, L.bytes);
  hipStream_t s = (hipStream_t)stream;
  PrArgs A;
  memset(&A, 0, sizeof(A));
  A.n = g->n;
  A.m = g->m;
  A.off = g->off;
  A.col = g->col;
  A.d = damping;
  A.base = (1.0 - damping) / (double)g->n;
  A.tol = tol;
  A.rank = rank;
  A.contrib[0] = L.contrib0;
  A.contrib[1] = L.contrib1;
  A.longrows = L.longrows;
  A.ctl = L.ctl;
  A.stats = stats;
  const fg_device_props pr = fg_props(g->device);
  A.clock_khz = pr.clock_khz;
  const int cus = pr.cus > 0 ? pr.cus : 256;
  PrPlanned Q;
  size_t loop_bytes;
  const size_t planned_bytes = pr_planned_layout(g, ws, &Q, &loop_bytes);
  if (max_iter >= (g->m <= PP_SMALL_M ? 2 : PP_MIN_ITER) && ws_bytes >= planned_bytes) {
    // one workgroup per CU (their LDS), a multiple of the column classes
    const int grid = cus >= PP_XCD ? cus / PP_XCD * PP_XCD : PP_XCD;
    int32_t longs = g->max_degree >= PP_SHORT;
    const bool loop = tol > 0.0 && pr.coop && ws_bytes >= loop_bytes;
    pp_clear_kernel<<<1, PP_BT, 0, s>>>(A, Q.plan, loop ? Q.bar : nullptr);
    pp_count_kernel<<<Q.tiles, PP_BT, 0, s>>>(g->n, g->off, Q);
    pp_prefix_kernel<<<PP_BUCKETS, PP_BT, 0, s>>>(Q);
    pp_scan_kernel<<<1, PP_SCAN_BT, 0, s>>>(g->m, Q.plan);
    pp_number_kernel<<<Q.tiles, PP_BT, 0, s>>>(g->n, g->off, Q, 1.0 / (double)g->n);
    pp_columns_kernel<<<grid, PP_BT, 0, s>>>(g->col, Q);
    if (loop) {
      void* args[] = {&A, &Q, &max_iter, &longs};
      FG_HIP_TRY(hipLaunchCooperativeKernel((const void*)pp_loop_kernel, dim3(grid), dim3(PP_BT),
                                            args, 0, s));
    } else {
      for (int32_t it = 0; it < max_iter; ++it) {
        if (longs) pp_long_kernel<<<grid, PP_BT, 0, s>>>(Q, it);
        pp_iter_kernel<<<grid, PP_BT, 0, s>>>(A, Q, it);
      }
    }
    pp_ranks_kernel<<<grid * 2, PP_BT, 0, s>>>(A, Q);
    FG_HIP_TRY(hipGetLastError());
    return FG_OK;
  }
  pr_reset_kernel<<<1, 64, 0, s>>>(L.ctl);
  pr_setup_kernel<<<cus * 4, PR_BT, 0, s>>>(A, 1.0 / (double)g->n);
  for (int32_t it = 0; it < max_iter; ++it) pr_iter_kernel<<<cus * 4, PR_BT, 0, s>>>(A, it);
  FG_HIP_TRY(hipGetLastError());
  return FG_OK;
}
