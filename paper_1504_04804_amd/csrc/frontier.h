// Device building blocks shared by the persistent traversal kernels
// (BFS and SSSP): padded counters, per-wave LDS staging of outputs, and the
// wave-level search used by the scan-gather expansion.
#pragma once

#include "fg_common.h"

namespace fgk {

typedef unsigned long long ull;

// Most entries are in rows far longer than the mean: the mean degree at an
// entry's end is at least twice that of a vertex (grids and uniform random
// graphs, whatever single hubs they have, 1.0 to 1.5 times; R-MAT 7 to 80,
// still 2.6 where a quarter of all pairs are edges).
static inline bool fg_skewed(const fg_graph* g) {
  return (double)g->deg_sq * (double)g->n >= 2.0 * (double)g->m * (double)g->m;
}

// Default width of a persistent launch: a grid barrier of 64 workgroups is 1
// to 2 us cheaper than one of 256 and so is their launch, which is worth more
// than the width where vertices and entries are few.  The bounds are each
// kernel's own (see its launch), where the wider launch catches up.
static inline int fg_default_width(const fg_graph* g, int64_t n64, int64_t n128, int64_t m64,
                                   int64_t m128, int full) {
  const int w = g->n <= n64 && g->m <= m64 ? 64 : g->n <= n128 && g->m <= m128 ? 128 : full;
  return w < full ? w : full;
}

// Pieces of `per` entries in a row (a row may have 2^31 - 1).
__host__ __device__ __forceinline__ int32_t fg_pieces(int32_t entries, int32_t per) {
  return (int32_t)(((uint32_t)entries + (uint32_t)per - 1u) / (uint32_t)per);
}

// One 256-byte line per counter so concurrent atomics do not share a line.
struct alignas(256) Line64 {
  ull v;
  ull pad[31];
};

// Entries are staged per wave in LDS and written out with one global atomic
// per batch, so concurrent waves do not serialise on the shared counter.
template <class T, int CAP>
struct WaveStage {
  T* buf;
  int32_t cnt;

  __device__ __forceinline__ void flush(ull* total, ull base, T* out) {
    if (cnt == 0) return;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    ull pos = 0;
    if (fg_lane() == 0) pos = atomicAdd(total, (ull)cnt);
    pos = __shfl(pos, 0, FG_WAVE) - base;
    // written through: read by other workgroups after the next barrier
    for (int i = fg_lane(); i < cnt; i += FG_WAVE) fg_st_shared(&out[pos + i], buf[i]);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    cnt = 0;
  }

  __device__ __forceinline__ void push(bool keep, const T& x, ull* total, ull base, T* out) {
    const uint64_t mask = __ballot(keep);
    if (!mask) return;
    const int32_t c = __popcll(mask);
    if (cnt + c > CAP) flush(total, base, out);
    if (keep) buf[cnt + fg_mbcnt(mask)] = x;
    cnt += c;
  }
};

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Largest j in [0, cnt) with sc[j] <= t (sc non-decreasing).
__device__ __forceinline__ int32_t upper_idx(const int32_t* sc, int32_t cnt, int32_t t) {
  int32_t lo = 0, hi = cnt - 1;
  while (lo < hi) {
    int32_t mid = (lo + hi + 1) >> 1;
    if (sc[mid] <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// End-of-phase flush of up to three kinds of staged entries by a workgroup of
// W waves: room for all waves' entries of a kind is reserved with one atomic
// per counter instead of one per wave.  Atomics on one address are served one
// after another (11.3 ns each), so the 4096 waves of a full launch otherwise
// spend 46 us per counter at the end of a phase, whatever the phase did.
template <int W>
struct FlushLds {
  int32_t cnt[3][W];
  ull pos[3];
};

// Positions of this wave's entries: pos[k] for the cnt[k] entries of kind k,
// reserved at ctr[k] (and counted at also[k] where that is not NULL).  Every
// thread of the workgroup calls it; cnt, ctr and also are wave-uniform.
template <int W, int K>
__device__ __forceinline__ void block_reserve(FlushLds<W>& F, const int32_t (&cnt)[K],
                                              ull* const (&ctr)[K], ull* const (&also)[K],
                                              ull (&pos)[K]) {
  const int lane = fg_lane();
  const int wid = threadIdx.x / FG_WAVE;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (lane == 0) F.cnt[k][wid] = cnt[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (wid != k) continue;
    // wave k reserves for kind k
    const int32_t c = lane < W ? F.cnt[k][lane] : 0;
    const int32_t incl = fg_wave_incl_scan(c);
    const int32_t all = __builtin_amdgcn_readlane(incl, FG_WAVE - 1);
    if (lane < W) F.cnt[k][lane] = incl - c;
    if (lane == 0) {
      F.pos[k] = all ? atomicAdd(ctr[k], (ull)all) : 0ull;
      if (all && also[k]) atomicAdd(also[k], (ull)all);
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) pos[k] = F.pos[k] + (ull)F.cnt[k][wid];
}

// Writes a wave's staged entries to out[pos - base ...] (written through:
// read by other workgroups after the next barrier) and empties the stage.
template <class S, class T>
__device__ __forceinline__ void put_staged(S& st, ull pos, ull base, T* out) {
  for (int i = fg_lane(); i < st.cnt; i += FG_WAVE) fg_st_shared(&out[pos - base + i], st.buf[i]);
  st.cnt = 0;
}

}  // namespace fgk
