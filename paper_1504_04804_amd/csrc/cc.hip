// Connected components (Table I's CC primitive; the hooking and
// pointer-jumping scheme of Soman et al. that the paper cites): every
// vertex is labelled with the smallest vertex id of its component.
//
// The label array itself holds a forest in which every vertex points to a
// smaller (or equal) vertex of its own component.  Hooking an edge {u, v}
// finds both roots (with path halving: the pointer jumping) and links the
// larger root under the smaller one by a compare-and-swap that succeeds
// only while it is still a root (a failed swap returns the new parent, from
// which the search continues).  Links only ever point to a smaller root, so
// the smallest vertex of a component is never linked and ends as the root
// of the whole component: the labels are the component minima whatever the
// order of the hooks.
//
// The order of the hooks is free, which the passes use (the neighbour
// sampling of Sutton, Ben-Nun and Barak's Afforest):
//   link     every vertex hooks its first two neighbours (the graph's head
//            table: one coalesced 16-byte load per vertex); on graphs with
//            hubs the first one while the labels are initialised, by
//            pointing the vertex at its first neighbour when that is
//            smaller (a forest already, no atomics)
//   compress every label becomes its root
//   sample   the most frequent root of 1024 sampled vertices, c: on graphs
//            with a giant component, that component's root
//   hook     every row of a vertex outside c's tree is hooked in full
//            (entries after the first two); rows of c's members are
//            skipped: each of their edges either stays inside c's tree or
//            is hooked from the other end's row
//   compress every label becomes its root (walks without re-pointing).
// The hook pass looks at every vertex once (label and degree, coalesced):
// where c is a giant component hardly any row is left, and a wave lays those
// of its 64 vertices end to end over its lanes.  Rows longer than CC_LONG
// outside c's tree, if there are any, get an edge-balanced pass of their
// own: tasks of CSR entries whose rows are found with a binary search over
// the offsets (staged in LDS).  Finding the rows of every task, with nothing
// to do in nearly all of them, took 168 us on R-MAT 22; the look at the
// vertices takes 8 us.
#include <string.h>

#include "fg_common.h"
#include "frontier.h"

namespace {

constexpr int CC_BT = 256;
constexpr int CC_TASK = 4096;           // CSR entries per workgroup task
constexpr int CC_LDS_OFF = 4096 + 2;    // offsets staged per task
constexpr int CC_SAMPLES = 1024;
constexpr int CC_CAND = FG_WAVE;        // samples that stand as candidates
constexpr int CC_SKIP = 2;              // entries per row hooked by the link pass
constexpr int CC_LONG = 64;             // longer rows are hooked by the edge-balanced pass
constexpr int CC_FINAL_BT = 1024;       // workgroup of the counting compress pass

struct CcCtl {
  int32_t giant;                // the sampled most frequent root
  int32_t longrows;             // set if a row past CC_LONG has to be hooked
  int64_t comps;                // the count, for an output that kernels cannot count in
};

// Root of x with path halving: each visited vertex is re-pointed at its
// grandparent.  A vertex only ever points to a smaller vertex of its own
// tree (stale reads included: trees only merge), so the walk always ends
// at a vertex that was a root when it was read.
__device__ __forceinline__ int32_t cc_find(int32_t* __restrict__ p, int32_t x) {
  int32_t cur = p[x];
  if (cur == x) return x;
  int32_t prev = x;
  int32_t next;
  while (cur > (next = p[cur])) {
    p[prev] = next;
    prev = cur;
    cur = next;
  }
  return cur;
}

// Joins the trees of a and b (hooking): the larger root goes under the
// smaller one while it is still a root.
__device__ __forceinline__ void cc_unite(int32_t* __restrict__ p, int32_t a, int32_t b) {
  int32_t ra = cc_find(p, a);
  int32_t rb = cc_find(p, b);
  while (ra != rb) {
    if (ra < rb) {
      const int32_t t = ra;
      ra = rb;
      rb = t;
    }
    const int32_t old = atomicCAS(&p[ra], ra, rb);
    if (old == ra) return;
    ra = cc_find(p, old);
  }
}

// Root of x without re-pointing (for passes that publish roots): once a
// vertex holds its root, a path-halving store from a walk that passed it
// earlier could put an intermediate vertex back.
__device__ __forceinline__ int32_t cc_root(const int32_t* p, int32_t x) {
  int32_t cur = p[x];
  while (cur != x) {
    x = cur;
    cur = p[x];
  }
  return cur;
}

// label[v] = v, or v's first neighbour where that one is smaller: already
// a forest of pointers to smaller vertices of the same component, written
// without atomics (the first link of the link pass).
__global__ __launch_bounds__(CC_BT) void cc_init_kernel(int32_t n, const int4* __restrict__ head,
                                                        int32_t* __restrict__ label,
                                                        CcCtl* __restrict__ ctl,
                                                        int64_t* __restrict__ comps) {
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
       v += (int64_t)gridDim.x * blockDim.x) {
    int32_t l = (int32_t)v;
    if (head) {
      const int32_t u = head[v].x;  // -1 without entries
      if (u >= 0 && u < l) l = u;
    }
    label[v] = l;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctl->giant = -1;
    ctl->longrows = 0;
    if (comps) *comps = 0;
  }
}

// Hooks from the head table: the first entry of every row (LINK_FIRST),
// the second (LINK_SECOND), or the second and, where the init pass did not
// link it (a first neighbour larger than the vertex), the first
// (LINK_REST).  After the passes run, both first entries of every row are
// hooked.
constexpr int LINK_FIRST = 0, LINK_SECOND = 1, LINK_REST = 2;
__global__ __launch_bounds__(CC_BT) void cc_link_kernel(int32_t n, const int4* __restrict__ head,
                                                        int32_t what, int32_t* __restrict__ label) {
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
       v += (int64_t)gridDim.x * blockDim.x) {
    const int4 h = head[v];
    // the head entry alone tells the rows apart: -1 without entries, the
    // second like the first with one (or twice the same, then one is enough)
    if (h.x < 0) continue;
    if (what != LINK_SECOND && (what == LINK_FIRST ? h.x != (int32_t)v : h.x > (int32_t)v))
      cc_unite(label, (int32_t)v, h.x);
    if (what != LINK_FIRST && h.y != h.x && h.y != (int32_t)v) cc_unite(label, (int32_t)v, h.y);
  }
}

// label[v] = root of v; counts the roots when `comps` is given, with one
// atomic per workgroup (the count is one address, 11 ns per atomic: with one
// per wave of 256-thread workgroups the pass took 105 us on R-MAT 22 instead
// of the 15 us it takes with 512 workgroups of 1024 threads).
template <int BT>
__global__ __launch_bounds__(BT) void cc_compress_kernel(int32_t n, int32_t* __restrict__ label,
                                                         int64_t* __restrict__ comps) {
  __shared__ int32_t s_red[BT / FG_WAVE];
  int32_t roots = 0;
  for (int64_t v = (int64_t)blockIdx.x * BT + threadIdx.x; v < n;
       v += (int64_t)gridDim.x * BT) {
    const int32_t r = cc_root(label, (int32_t)v);
    label[v] = r;
    roots += r == (int32_t)v;
  }
  if (!comps) return;
  roots = fg_block_sum<BT>(roots, s_red);
  if (threadIdx.x == 0 && roots)
    atomicAdd((unsigned long long*)comps, (unsigned long long)roots);
}

// The most frequent, among CC_SAMPLES spread-out vertices, of the labels of
// the first CC_CAND of them (one workgroup; ties go to the smaller label): a
// component that holds a tenth of the vertices is missed once in 800 graphs,
// and then only the hook pass has more to do.  Every wave compares its
// samples with the candidates, one candidate per lane (comparing each sample
// with all others took 21 us).
__global__ __launch_bounds__(CC_SAMPLES) void cc_sample_kernel(int32_t n,
                                                               const int32_t* __restrict__ label,
                                                               CcCtl* __restrict__ ctl) {
  __shared__ int32_t s_cand[CC_CAND];
  __shared__ int32_t s_cnt[CC_CAND];
  const int t = threadIdx.x;
  const int lane = fg_lane();
  const uint64_t v = ((uint64_t)t * 0x9E3779B97F4A7C15ull + 0x5851F42D4C957F2Dull) % (uint64_t)n;
  const int32_t mine = label[v];
  if (t < CC_CAND) {
    s_cand[t] = mine;
    s_cnt[t] = 0;
  }
  __syncthreads();
  const int32_t cand = s_cand[lane];
  int32_t cnt = 0;
#pragma unroll
  for (int j = 0; j < FG_WAVE; ++j) cnt += __builtin_amdgcn_readlane(mine, j) == cand;
  atomicAdd(&s_cnt[lane], cnt);
  __syncthreads();
  if (t >= FG_WAVE) return;
  // key: count high, then the smaller label
  unsigned long long key =
      ((unsigned long long)s_cnt[lane] << 32) | (uint32_t)(0x7fffffff - cand);
  for (int s = FG_WAVE / 2; s > 0; s >>= 1) {
    const unsigned long long o = __shfl_xor(key, s, FG_WAVE);
    key = o > key ? o : key;
  }
  if (t == 0) ctl->giant = 0x7fffffff - (int32_t)(uint32_t)key;
}

// Hooks the rows (of up to CC_LONG entries) of every vertex outside the
// sampled tree: a wave takes 64 vertices, lays the rows that have entries
// past the first two end to end and hooks 64 entries per step (so CC_LONG
// bounds a wave's steps; with rows of up to 1024 two cliques of 1000 vertices
// took 870 us, 50 of them 1056, two R-MAT graphs of 512 k vertices side by side
// 719: 32, 199 and 181 with 64; 128 and 256 are equal or slower).
__global__ __launch_bounds__(CC_BT) void cc_hook_rows_kernel(int32_t n,
                                                             const int32_t* __restrict__ off,
                                                             const int32_t* __restrict__ col,
                                                             int32_t* __restrict__ label,
                                                             CcCtl* __restrict__ ctl) {
  __shared__ int32_t s_sc[CC_BT / FG_WAVE][FG_WAVE];
  __shared__ int2 s_row[CC_BT / FG_WAVE][FG_WAVE];  // vertex, first entry to hook
  const int lane = fg_lane();
  const int wid = threadIdx.x / FG_WAVE;
  int32_t* sc = s_sc[wid];
  int2* row = s_row[wid];
  const int32_t giant = ctl->giant;
  const int64_t nth = (int64_t)gridDim.x * CC_BT;
  for (int64_t v0 = (int64_t)blockIdx.x * CC_BT + threadIdx.x - lane; v0 < n; v0 += nth) {
    const int64_t v = v0 + lane;
    int32_t b = 0, d = 0;
    if (v < n && label[v] != giant) {
      b = off[v];
      d = off[v + 1] - b;
    }
    if (d > CC_LONG) {
      ctl->longrows = 1;
      d = 0;
    }
    d = d > CC_SKIP ? d - CC_SKIP : 0;
    if (!__ballot(d > 0)) continue;
    const int32_t incl = fg_wave_incl_scan(d);
    const int32_t T = __builtin_amdgcn_readlane(incl, FG_WAVE - 1);
    fgk::wave_lds_fence();  // the lanes' reads of the step before are done
    sc[lane] = incl - d;
    row[lane] = make_int2((int32_t)v, b + CC_SKIP);
    fgk::wave_lds_fence();
    for (int32_t t = lane; t < T; t += FG_WAVE) {
      const int32_t j = fgk::upper_idx(sc, FG_WAVE, t);
      const int2 r = row[j];
      const int32_t u = col[r.y + (t - sc[j])];
      if (u != r.x) cc_unite(label, r.x, u);
    }
  }
}

// Largest u in [lo, hi] with off[u] <= e.
__device__ __forceinline__ int32_t row_of(const int32_t* __restrict__ off, int32_t lo, int32_t hi,
                                          int64_t e) {
  while (lo < hi) {
    const int32_t mid = lo + ((hi - lo + 1) >> 1);
    if ((int64_t)off[mid] <= e) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Hooks the rows past CC_LONG entries outside the sampled tree, if the pass
// over the vertices met one: edge-balanced, so a row of any length costs its
// share of the tasks.
__global__ __launch_bounds__(CC_BT) void cc_hook_kernel(int32_t n, int64_t m,
                                                        const int32_t* __restrict__ off,
                                                        const int32_t* __restrict__ col,
                                                        int32_t* __restrict__ label,
                                                        const CcCtl* __restrict__ ctl) {
  __shared__ int32_t s_off[CC_LDS_OFF];
  __shared__ int32_t s_u0, s_u1;
  if (!ctl->longrows) return;
  const int32_t giant = ctl->giant;
  const int64_t ntasks = (m + CC_TASK - 1) / CC_TASK;
  for (int64_t t = blockIdx.x; t < ntasks; t += gridDim.x) {
    const int64_t e0 = t * CC_TASK;
    const int64_t e1 = (e0 + CC_TASK < m ? e0 + CC_TASK : m);
    __syncthreads();
    if (threadIdx.x == 0) {
      // rows holding entries e0 and e1 - 1 (rows with no entries are skipped
      // by the search: it returns the last row starting at or before e)
      s_u0 = row_of(off, 0, n - 1, e0);
      s_u1 = row_of(off, s_u0, n - 1, e1 - 1);
    }
    __syncthreads();
    const int32_t u0 = s_u0, u1 = s_u1;
    const int32_t span = u1 - u0 + 2;  // offsets u0 .. u1 + 1
    const bool staged = span <= CC_LDS_OFF;
    if (staged)
      for (int32_t i = threadIdx.x; i < span; i += CC_BT) s_off[i] = off[u0 + i];
    __syncthreads();
    // a task without such a row has nothing to hook: one look at each row
    // instead of a search per entry
    int todo = 0;
    for (int32_t i = threadIdx.x; i <= u1 - u0 && !todo; i += CC_BT) {
      const int32_t u = u0 + i;
      const int32_t deg = staged ? s_off[i + 1] - s_off[i] : off[u + 1] - off[u];
      todo = deg > CC_LONG && label[u] != giant;
    }
    if (!__syncthreads_or(todo)) continue;
    for (int64_t e = e0 + threadIdx.x; e < e1; e += CC_BT) {
      int32_t u, first, end;
      if (staged) {
        int32_t lo = 0, hi = u1 - u0;
        while (lo < hi) {
          const int32_t mid = (lo + hi + 1) >> 1;
          if ((int64_t)s_off[mid] <= e) lo = mid; else hi = mid - 1;
        }
        u = u0 + lo;
        first = s_off[lo];
        end = s_off[lo + 1];
      } else {
        u = row_of(off, u0, u1, e);
        first = off[u];
        end = off[u + 1];
      }
      if (end - first <= CC_LONG) continue;   // hooked by the pass over the vertices
      if (e - first < CC_SKIP) continue;      // hooked by the link pass
      if (label[u] == giant) continue;        // a member of the sampled tree
      const int32_t v = col[e];
      if (v != u) cc_unite(label, u, v);
    }
  }
}

}  // namespace

size_t fg_cc_workspace_bytes(const fg_graph*) { return fg_align(sizeof(CcCtl)); }

extern "C" fg_status fg_cc(const fg_graph* g, int32_t* label, int64_t* components, void* ws,
                           size_t ws_bytes, void* stream) {
  if (!g || !label || !ws) return fg_set_error(FG_EINVAL, "fg_cc: NULL argument");
  if (!g->symmetric)
    return fg_set_error(FG_EUNSUPPORTED, "fg_cc: needs an undirected graph (FG_SYMMETRIC)");
  FG_CHECK_WS_ALIGN(ws, "fg_cc");
  if (ws_bytes < sizeof(CcCtl))
    return fg_set_error(FG_ENOMEM, "fg_cc: workspace of %zu bytes < required %zu", ws_bytes,
                        sizeof(CcCtl));
  hipStream_t s = (hipStream_t)stream;
  CcCtl* ctl = (CcCtl*)ws;
  int64_t* const comps =
      !components || (!((uintptr_t)components & 7) && fg_own_memory(components, g->device))
          ? components
          : &ctl->comps;
  const int cus = fg_props(g->device).cus;
  const int grid = (cus > 0 ? cus : 256) * 8;
  // On graphs with hubs (mean degree above 8) a vertex's first neighbour is
  // usually a smaller hub, and the init pass links it for free; on grids
  // and road-like graphs that would chain every vertex to the one before
  // it, so they hook both first entries by compare-and-swap.
  const bool init_link = g->m > 8 * (int64_t)g->n;
  cc_init_kernel<<<grid, CC_BT, 0, s>>>(g->n, init_link ? g->head : nullptr, label, ctl,
                                         comps);
  if (g->m > 0) {
    if (init_link) {
      cc_link_kernel<<<grid, CC_BT, 0, s>>>(g->n, g->head, LINK_REST, label);
    } else {
      cc_link_kernel<<<grid, CC_BT, 0, s>>>(g->n, g->head, LINK_FIRST, label);
      cc_link_kernel<<<grid, CC_BT, 0, s>>>(g->n, g->head, LINK_SECOND, label);
    }
    cc_compress_kernel<CC_BT><<<grid, CC_BT, 0, s>>>(g->n, label, nullptr);
    cc_sample_kernel<<<1, CC_SAMPLES, 0, s>>>(g->n, label, ctl);
    cc_hook_rows_kernel<<<grid, CC_BT, 0, s>>>(g->n, g->off, g->col, label, ctl);
    if (g->max_degree > CC_LONG)
      cc_hook_kernel<<<grid, CC_BT, 0, s>>>(g->n, g->m, g->off, g->col, label, ctl);
  }
  cc_compress_kernel<CC_FINAL_BT><<<grid / 4, CC_FINAL_BT, 0, s>>>(g->n, label, comps);
  if (comps != components)
    FG_HIP_TRY(hipMemcpyAsync(components, comps, sizeof(int64_t), hipMemcpyDeviceToDevice, s));
  FG_HIP_TRY(hipGetLastError());
  return FG_OK;
}
