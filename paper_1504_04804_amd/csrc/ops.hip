// Standalone frontier operators (Sec. II-B): advance with a deterministic
// edge-frontier layout, filter with the visited test-and-set, one backward
// (pull) step (Sec. VI-A), queue <-> bitmap conversions, and the unfused
// push BFS that chains advance and filter kernels (Alg. 1 as an advance
// kernel followed by a filter kernel).
#include <string.h>

#include <vector>

#include "fg_common.h"

namespace {

constexpr int TB = 1024;          // tile of the scans (one block, one element per thread)
constexpr int EXP_PER_BLOCK = 2048;

// ------------------------------------------------------------ scan helpers

// Up to this many tiles a scan's second kernel sums the tile sums before its
// own tile itself (at most two loads per thread, eight in tiles of 256), which
// saves the one-block kernel in between; above it that kernel scans them once.  A launch that has
// nothing to do costs about 4.8 us in a chain of dependent kernels; 2048
// tiles read 16 MB of sums from the L2s in all, under that.
constexpr int SELF_TILES = 2048;
constexpr int QB = 256;  // words per tile of bitmap -> queue (smaller: 64 words a wave to write)

// Block sums of `val(i)` over tiles of BT elements.
template <int BT, class F>
__global__ void tile_sum_kernel(int64_t len, F val, int64_t* __restrict__ sums) {
  __shared__ int64_t red[BT / FG_WAVE + 1];
  const int64_t i = (int64_t)blockIdx.x * BT + threadIdx.x;
  int64_t x = i < len ? val(i) : 0;
  int64_t s = fg_block_sum<BT>(x, red);
  if (threadIdx.x == 0) sums[blockIdx.x] = s;
}

// Exclusive scan of `cnt` tile sums in place (single block), total -> *total.
__global__ void scan_sums_kernel(int64_t cnt, int64_t* __restrict__ sums,
                                 int64_t* __restrict__ total) {
  __shared__ int64_t red[TB / FG_WAVE + 1];
  int64_t carry = 0;
  for (int64_t c0 = 0; c0 < cnt; c0 += TB) {
    const int64_t i = c0 + threadIdx.x;
    int64_t x = i < cnt ? sums[i] : 0;
    int64_t tot = 0;
    int64_t ex = fg_block_excl_scan<TB>(x, red, &tot);
    if (i < cnt) sums[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) *total = carry;
}

// The sum of everything before this block's tile: the scanned tile sum, or
// (SELF) the sum of the raw tile sums before it.
template <bool SELF, int BT>
__device__ __forceinline__ int64_t tile_base(const int64_t* sums, int64_t* red) {
  if (!SELF) return sums[blockIdx.x];
  int64_t x = 0;
  for (unsigned j = threadIdx.x; j < blockIdx.x; j += BT) x += sums[j];
  return fg_block_sum<BT>(x, red);
}

// Exclusive scan of val(i) from the tile sums; out[i] for i < len.  With
// SELF the last tile also writes the total.
template <bool SELF, class F>
__global__ void tile_scan_kernel(int64_t len, F val, const int64_t* __restrict__ sums,
                                 int64_t* __restrict__ out, int64_t* __restrict__ total) {
  __shared__ int64_t red[TB / FG_WAVE + 1];
  const int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x;
  int64_t x = i < len ? val(i) : 0;
  const int64_t base = tile_base<SELF, TB>(sums, red);
  int64_t tot = 0;
  int64_t ex = fg_block_excl_scan<TB>(x, red, &tot);
  if (i < len) out[i] = base + ex;
  if (SELF && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = base + tot;
}

// Degree of frontier entry i; entries at or past the device-resident
// length *dlen (when given) count as degree 0.
struct DegOf {
  const int32_t* off;
  const int32_t* q;
  const int32_t* dlen;
  __device__ int64_t operator()(int64_t i) const {
    if (dlen && i >= (int64_t)*dlen) return 0;
    int32_t u = q[i];
    return (int64_t)(off[u + 1] - off[u]);
  }
};

struct PopOf {
  const uint64_t* bits;
  __device__ int64_t operator()(int64_t i) const { return __popcll(bits[i]); }
};

// Scan workspace: tile sums + scanned values + total.
struct ScanWs {
  int64_t* sums;   // ceil(len / TB)
  int64_t* scan;   // len
  int64_t* total;  // 1
};

template <class F>
void run_scan(int64_t len, F f, ScanWs w, hipStream_t s) {
  const int64_t tiles = (len + TB - 1) / TB;
  if (tiles > 0) tile_sum_kernel<TB><<<(unsigned)tiles, TB, 0, s>>>(len, f, w.sums);
  if (tiles > 0 && tiles <= SELF_TILES) {
    tile_scan_kernel<true><<<(unsigned)tiles, TB, 0, s>>>(len, f, w.sums, w.scan, w.total);
    return;
  }
  scan_sums_kernel<<<1, TB, 0, s>>>(tiles, w.sums, w.total);
  if (tiles > 0)
    tile_scan_kernel<false><<<(unsigned)tiles, TB, 0, s>>>(len, f, w.sums, w.scan, w.total);
}

// -------------------------------------------------------------- advance

// Largest i in [lo, hi] with scan[i] <= t.
__device__ __forceinline__ int64_t scan_upper(const int64_t* scan, int64_t lo, int64_t hi,
                                              int64_t t) {
  while (lo < hi) {
    int64_t mid = (lo + hi + 1) >> 1;
    if (scan[mid] <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// The same by a whole wave, 64 probes per step (every lane calls it with the
// same arguments and gets the result): three dependent loads where the
// halving search of one lane takes sixteen, which made the expansion of 1.1 M edges
// 21 us (16 us now).
__device__ __forceinline__ int64_t wave_scan_upper(const int64_t* scan, int64_t lo, int64_t hi,
                                                   int64_t t) {
  const int lane = fg_lane();
  while (lo < hi) {
    const int64_t step = (hi - lo + FG_WAVE - 1) / FG_WAVE;
    const int64_t at = lo + (lane + 1) * step;  // probes ascend; those past hi count as greater
    const int c = __popcll(__ballot(at <= hi && scan[at <= hi ? at : hi] <= t));
    const int64_t top = lo + (c + 1) * step - 1;
    lo += c * step;
    hi = top < hi ? top : hi;
  }
  return lo;
}

// Each block writes EXP_PER_BLOCK consecutive slots of the edge frontier.
// Slot t belongs to frontier entry i = last index with scan[i] <= t.
__global__ void advance_expand_kernel(int64_t len, const int32_t* __restrict__ q,
                                      const int32_t* __restrict__ off,
                                      const int32_t* __restrict__ col,
                                      const int64_t* __restrict__ scan,
                                      const int64_t* __restrict__ total, int64_t capacity,
                                      int32_t* __restrict__ out_dst,
                                      int32_t* __restrict__ out_src,
                                      int64_t* __restrict__ out_len) {
  __shared__ int64_t s_scan[EXP_PER_BLOCK + 1];
  __shared__ int64_t s_lo, s_hi;
  const int64_t T = *total;
  if (blockIdx.x == 0 && threadIdx.x == 0 && out_len) *out_len = T;
  const int64_t lim = T < capacity ? T : capacity;
  for (int64_t t0 = (int64_t)blockIdx.x * EXP_PER_BLOCK; t0 < lim;
       t0 += (int64_t)gridDim.x * EXP_PER_BLOCK) {
    const int64_t t1 = (t0 + EXP_PER_BLOCK < lim ? t0 + EXP_PER_BLOCK : lim) - 1;
    __syncthreads();
    const int wid = threadIdx.x / FG_WAVE;
    if (wid < 2) {  // the first and the last entry of the slots, a wave each
      const int64_t x = wave_scan_upper(scan, 0, len - 1, wid == 0 ? t0 : t1);
      if (fg_lane() == 0) (wid == 0 ? s_lo : s_hi) = x;
    }
    __syncthreads();
    const int64_t lo = s_lo, cnt = s_hi - lo + 1;
    const bool in_lds = cnt <= EXP_PER_BLOCK + 1;
    if (in_lds)
      for (int64_t j = threadIdx.x; j < cnt; j += blockDim.x) s_scan[j] = scan[lo + j];
    __syncthreads();
    for (int64_t t = t0 + threadIdx.x; t <= t1; t += blockDim.x) {
      int64_t i;
      if (in_lds) {
        int64_t a = 0, b = cnt - 1;
        while (a < b) {
          int64_t mid = (a + b + 1) >> 1;
          if (s_scan[mid] <= t) a = mid; else b = mid - 1;
        }
        i = lo + a;
      } else {
        i = scan_upper(scan, lo, lo + cnt - 1, t);
      }
      const int32_t u = q[i];
      const int64_t base = in_lds ? s_scan[i - lo] : scan[i];
      out_dst[t] = col[off[u] + (t - base)];
      out_src[t] = u;
    }
  }
}

// ------------------------------------------------ staged appends to a queue

// A workgroup collects what it appends to the output queue in LDS and
// reserves room for all of it with one atomic: the queue's counter is one
// address for the whole launch, and atomics on one address are served one
// after another, 11.3 ns each.
template <int BT, int CAP>
struct BlockStage {
  int32_t* buf;   // LDS, CAP entries
  int32_t* cnt;   // LDS
  int32_t* base;  // LDS

  // Appends the calling wave's kept lanes (at most CAP minus what is staged,
  // which the caller ensures by its flushes).
  __device__ __forceinline__ void push(bool keep, int32_t v) {
    const uint64_t mask = __ballot(keep);
    if (!mask) return;
    int32_t pos = 0;
    if (fg_lane() == 0) pos = atomicAdd(cnt, __popcll(mask));
    pos = __builtin_amdgcn_readfirstlane(pos);
    if (keep) buf[pos + fg_mbcnt(mask)] = v;
  }

  // Writes the staged entries out if more than `most` are staged.  Every
  // thread of the workgroup calls it with the same `most`, after a barrier
  // that follows the last push; pushes may follow at once (every thread has
  // read the count by then).
  __device__ __forceinline__ void flush_above(int32_t most, int32_t* out_q, int32_t* out_len) {
    const int32_t c = *cnt;
    __syncthreads();
    if (c <= most) return;
    if (threadIdx.x == 0) *base = atomicAdd(out_len, c);
    __syncthreads();
    const int32_t b = *base;
    for (int32_t i = threadIdx.x; i < c; i += BT) out_q[b + i] = buf[i];
    if (threadIdx.x == 0) *cnt = 0;
    __syncthreads();
  }
};

// --------------------------------------------------------------- filter

__global__ void fill_i32_kernel(int32_t* p, int64_t count, int32_t value) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = value;
}

constexpr int FT_BT = 1024;
constexpr int FT_R = 8;                  // edges per thread and tile
constexpr int FT_TILE = FT_BT * FT_R;
constexpr int FT_STAGE = FT_TILE;
constexpr int FT_SLOTS = 4096;           // visited words a tile combines
constexpr int FT_SPREAD = 128;           // tiles from which a tile takes more per thread
constexpr int FT_ONCE = 2;               // edges per thread up to which one round is enough

// A word's slot: neighbouring words lie in neighbouring slots, and words 4096
// apart (an R-MAT graph's hubs, a wide grid's column) in unrelated ones.
__device__ __forceinline__ int ft_slot(int32_t word) {
  return (int)((uint32_t)word ^ (((uint32_t)word >> 12) * 0x9E3779B1u >> 20)) & (FT_SLOTS - 1);
}

// Test-and-set of dst's visited bit; winners take depth / parent and are
// appended to out_q.  The edge-frontier length is read from device memory
// (`d_len`, clamped to `cap`) or taken from `h_len` when d_len is NULL.
//
// Atomics on one word are served one after another at the point of
// coherence (11.3 ns each; 0.04 ns where the words lie in different lines,
// 0.007 ns for consecutive words), and a scale-free edge frontier repeats
// its hubs' few words: with one test-and-set per edge whose vertex looked
// unvisited the kernel took 279 us on 1.1 M edges (R-MAT of 1 M vertices).
// So a workgroup combines a tile first: its bits go into a direct-mapped
// LDS table of visited words (ft_slot; of two words in one slot the one whose
// edge wrote last, most likely the busier, keeps it), one atomic per word takes
// them to memory, neighbouring slots by neighbouring lanes, and the edge that
// set a bit in the table first wins the vertex if memory says the bit is new.
// Words that lost their slot get a second round in full tiles; what is left
// then is tested in memory by itself.  On the 1.1 M edges that takes 36 us (one
// round 43, three 37, rounds until nothing is left 42; with a slot that is the
// word's id modulo FT_SLOTS and rounds to the end 62, and 1360 us on 512 words
// 4096 apart, 12 here).  Short lists are spread over FT_SPREAD tiles (15 k
// edges 10 us, as with a test per edge; one tile of 8192 edges after another
// took 60), long ones need full tiles: the hot lines get one request per tile
// and round.  The look before that reads past the caches (agent scope), so
// vertices that other workgroups have set meanwhile are not tried again.
__global__ __launch_bounds__(FT_BT) void filter_kernel(
    const int32_t* __restrict__ dst, const int32_t* __restrict__ src,
    const int64_t* __restrict__ d_len, int64_t h_len, int64_t cap,
    uint32_t* __restrict__ visited, int32_t d_new, int32_t* __restrict__ depth,
    int32_t* __restrict__ parent, int32_t* __restrict__ out_q, int32_t* __restrict__ out_len) {
  __shared__ int32_t s_buf[FT_STAGE];
  __shared__ int32_t s_tag[FT_SLOTS];
  __shared__ uint32_t s_bits[FT_SLOTS];
  __shared__ int32_t s_cnt, s_base;
  int64_t len = d_len ? *d_len : h_len;
  if (len > cap) len = cap;
  const int64_t fair = (len + (int64_t)FT_SPREAD * FT_BT - 1) / ((int64_t)FT_SPREAD * FT_BT);
  const int per = fair < FT_R ? (int)fair : FT_R;  // edges per thread and tile
  const int64_t tile = (int64_t)per * FT_BT;
  if ((int64_t)blockIdx.x * tile >= len) return;  // the whole workgroup
  BlockStage<FT_BT, FT_STAGE> stage{s_buf, &s_cnt, &s_base};
  if (threadIdx.x == 0) s_cnt = 0;
  for (int64_t t0 = (int64_t)blockIdx.x * tile; t0 < len; t0 += (int64_t)gridDim.x * tile) {
    int32_t v[FT_R];
    uint32_t word[FT_R];
    bool open[FT_R];
#pragma unroll
    for (int r = 0; r < FT_R; ++r) {
      const int64_t k = t0 + r * FT_BT + threadIdx.x;
      v[r] = r < per && k < len ? dst[k] : -1;
    }
#pragma unroll
    for (int r = 0; r < FT_R; ++r)
      word[r] = v[r] >= 0 ? fg_atomic_load_u32(&visited[v[r] >> 5]) : ~0u;
    bool any = false;
#pragma unroll
    for (int r = 0; r < FT_R; ++r) {
      open[r] = !((word[r] >> (v[r] & 31)) & 1u);
      any = any || open[r];
    }
    for (int round = per <= FT_ONCE ? 1 : 2; round > 0 && __syncthreads_or(any); --round) {
      for (int i = threadIdx.x; i < FT_SLOTS; i += FT_BT) s_bits[i] = 0;
#pragma unroll
      for (int r = 0; r < FT_R; ++r)
        if (open[r]) s_tag[ft_slot(v[r] >> 5)] = v[r] >> 5;
      __syncthreads();
      bool first[FT_R];
      any = false;
#pragma unroll
      for (int r = 0; r < FT_R; ++r) {
        const int slot = ft_slot(v[r] >> 5);
        const uint32_t bit = 1u << (v[r] & 31);
        first[r] = open[r] && s_tag[slot] == v[r] >> 5;
        open[r] = open[r] && !first[r];
        // an edge that is not the first of its vertex here is done
        if (first[r]) first[r] = !(atomicOr(&s_bits[slot], bit) & bit);
        any = any || open[r];
      }
      __syncthreads();
      for (int i = threadIdx.x; i < FT_SLOTS; i += FT_BT) {
        const uint32_t mine = s_bits[i];
        if (mine) s_bits[i] = mine & ~atomicOr(&visited[s_tag[i]], mine);
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < FT_R; ++r) {
        const bool won =
            first[r] && ((s_bits[ft_slot(v[r] >> 5)] >> (v[r] & 31)) & 1u);
        if (won) {
          depth[v[r]] = d_new;
          if (parent) parent[v[r]] = src[t0 + r * FT_BT + threadIdx.x];
        }
        stage.push(won, v[r]);
      }
    }
    // what is left by itself: words that were always beside a busier one
#pragma unroll
    for (int r = 0; r < FT_R; ++r)
      word[r] = open[r] ? fg_atomic_load_u32(&visited[v[r] >> 5]) : ~0u;
#pragma unroll
    for (int r = 0; r < FT_R; ++r) {
      const uint32_t bit = 1u << (v[r] & 31);
      open[r] = open[r] && !(word[r] & bit);
      if (open[r]) word[r] = atomicOr(&visited[v[r] >> 5], bit);
    }
#pragma unroll
    for (int r = 0; r < FT_R; ++r) {
      const bool won = open[r] && !((word[r] >> (v[r] & 31)) & 1u);
      if (won) {
        depth[v[r]] = d_new;
        if (parent) parent[v[r]] = src[t0 + r * FT_BT + threadIdx.x];
      }
      stage.push(won, v[r]);
    }
    __syncthreads();
    stage.flush_above(FT_STAGE - FT_TILE, out_q, out_len);
  }
  stage.flush_above(0, out_q, out_len);
}

// ------------------------------------------------------------ pull step

constexpr int PL_BT = 512;
constexpr int PL_WAVES = PL_BT / FG_WAVE;
constexpr int PL_STAGE = 2 * PL_BT;
constexpr int PL_GRID = 1021;    // workgroups at most (odd, see below)
constexpr int PL_LANE = 32;      // rows up to this length are scanned by their lane
constexpr int PL_GROUP = 16;     // lanes that scan a longer row together ...
constexpr int PL_GROUP_MAX = 260;  // ... up to this entry; the rest by a wave

__device__ __forceinline__ bool bit_of(const uint32_t* bits, int32_t u) {
  return (bits[u >> 5] >> (u & 31)) & 1u;
}

// The first entry from `c` on, of `width` lanes times four, whose bit is set:
// its place from c (-1 = none) in *at and its vertex in *got.  The lanes of
// a group pass the same c and end; `first` is the group's first lane.  A
// group without a row passes c >= end.
__device__ __forceinline__ void probe_row(const int32_t* col, const uint32_t* fbits, uint32_t c,
                                          uint32_t end, int first, int width, int32_t* at,
                                          int32_t* got) {
  const int lane = fg_lane();
  int32_t u[4];
  bool hit[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint32_t k = c + r * width + (lane - first);
    u[r] = k < end ? col[k] : -1;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) hit[r] = u[r] >= 0 && bit_of(fbits, u[r]);
  const uint64_t group = (width == FG_WAVE ? ~0ull : ((1ull << width) - 1ull)) << first;
  *at = -1;
#pragma unroll
  for (int r = 3; r >= 0; --r) {
    const uint64_t m = __ballot(hit[r]) & group;
    const int l = m ? __builtin_ctzll(m) : first;
    const int32_t x = __shfl(u[r], l, FG_WAVE);
    if (m) {
      *at = r * width + (l - first);
      *got = x;
    }
  }
}

// Places in the columns are unsigned: one past a row's end may pass 2^31 - 1.
// One early-exit backward step: a lane per unvisited vertex of nonzero
// degree.  The first four entries come from the head table (one coalesced
// load instead of a random line per vertex); rows of up to PL_LANE entries
// go on four at a time in their lane; longer rows are listed and taken by
// groups of 16 lanes, 64 entries per step and four rows per wave, and what
// is still open after 256 more by whole waves, 256 entries per step.  The
// entries of a step are loaded together and counted up to the first hit, so
// `inspected` is the early-exit count.
// Bound by the latency of the dependent loads (column, then frontier word):
// a step takes about 1.5 us whatever its width, so the rows in flight
// count, and a workgroup takes words from all over the graph (word
// blockIdx + j gridDim) because long rows lie together.  The largest grid is
// odd: an R-MAT vertex's degree follows the bits of its id, and with 512
// workgroups those whose words end in zeros took four times as long.
// R-MAT of 1 M vertices, frontier of 2 %: 229 us with a lane per row and an
// atomic per wave for each counter, 210 us with rows past 32 entries given
// to waves one at a time, 89 us in groups of 16 lanes, 55 us with the words
// spread and 512 threads (8 words) per workgroup.
__global__ __launch_bounds__(PL_BT) void pull_step_kernel(
    int32_t nwords, const int32_t* __restrict__ off, const int32_t* __restrict__ col,
    const int4* __restrict__ head, const uint64_t* __restrict__ nz,
    const uint32_t* __restrict__ fbits, uint64_t* __restrict__ visited,
    uint64_t* __restrict__ next_bits, int32_t d_new, int32_t* __restrict__ depth,
    int32_t* __restrict__ parent, int32_t* __restrict__ out_q, int32_t* __restrict__ out_len,
    int64_t* __restrict__ inspected) {
  __shared__ int32_t s_buf[PL_STAGE];
  __shared__ int2 s_long[PL_BT];  // vertex, wave of this workgroup that holds its word
  __shared__ int2 s_hub[PL_BT];
  __shared__ unsigned long long s_new[PL_WAVES];
  __shared__ int64_t s_red[PL_WAVES + 1];
  __shared__ int32_t s_cnt, s_base, s_nlong, s_nhub;
  BlockStage<PL_BT, PL_STAGE> stage{s_buf, &s_cnt, &s_base};
  const int lane = fg_lane();
  const int wid = threadIdx.x / FG_WAVE;
  if (threadIdx.x == 0) s_cnt = 0;
  int64_t insp = 0;
  for (int64_t w0 = blockIdx.x; w0 < nwords; w0 += (int64_t)gridDim.x * PL_WAVES) {
    const int64_t w = w0 + (int64_t)wid * gridDim.x;
    const uint64_t vis = w < nwords ? visited[w] : ~0ull;
    const uint64_t act = w < nwords ? nz[w] & ~vis : 0ull;
    if (threadIdx.x == 0) s_nlong = s_nhub = 0;
    __syncthreads();
    const int32_t v = (int32_t)(w * 64 + lane);
    uint32_t i = 0, e = 0;
    int32_t pu = -1;
    bool open = (act >> lane) & 1ull;
    bool found = false;
    if (open) {
      i = off[v];
      e = off[v + 1];
      const int4 h = head[v];
      const bool h0 = bit_of(fbits, h.x), h1 = bit_of(fbits, h.y);
      const bool h2 = bit_of(fbits, h.z), h3 = bit_of(fbits, h.w);
      // entries past the degree repeat the last one: a hit there is a hit
      // of the last entry, found first
      const int32_t d = e - i < 4 ? e - i : 4;
      found = h0 || h1 || h2 || h3;
      pu = h0 ? h.x : h1 ? h.y : h2 ? h.z : h.w;
      insp += h0 ? 1 : h1 ? 2 : h2 ? 3 : d;
      i += 4;
      open = !found && i < e;
    }
    {
      const bool listed = open && e - i > PL_LANE - 4;
      const uint64_t mask = __ballot(listed);
      if (mask) {
        int32_t pos = 0;
        if (lane == 0) pos = atomicAdd(&s_nlong, __popcll(mask));
        pos = __builtin_amdgcn_readfirstlane(pos);
        if (listed) s_long[pos + fg_mbcnt(mask)] = make_int2(v, wid);
        open = open && !listed;
      }
    }
    while (__ballot(open)) {
      if (open) {
        const uint32_t l = e - 1;
        const int32_t u0 = col[i], u1 = col[i + 1 < l ? i + 1 : l];
        const int32_t u2 = col[i + 2 < l ? i + 2 : l], u3 = col[i + 3 < l ? i + 3 : l];
        const bool h0 = bit_of(fbits, u0), h1 = bit_of(fbits, u1);
        const bool h2 = bit_of(fbits, u2), h3 = bit_of(fbits, u3);
        const int32_t d = e - i < 4 ? e - i : 4;
        found = h0 || h1 || h2 || h3;
        pu = h0 ? u0 : h1 ? u1 : h2 ? u2 : u3;
        insp += h0 ? 1 : h1 ? 2 : h2 ? 3 : d;
        i += 4;
        open = !found && i < e;
      }
    }
    {
      const uint64_t nb = __ballot(found);
      if (lane == 0) s_new[wid] = nb;
    }
    if (found) {
      depth[v] = d_new;
      if (parent) parent[v] = pu;
    }
    stage.push(found, v);
    __syncthreads();
    const int32_t nlong = s_nlong;
    for (int32_t j0 = wid * (FG_WAVE / PL_GROUP); j0 < nlong; j0 += PL_BT / PL_GROUP) {
      const int first = lane & ~(PL_GROUP - 1);
      const int32_t j = j0 + lane / PL_GROUP;
      int2 x = make_int2(0, 0);
      uint32_t c = 0, end = 0;
      if (j < nlong) {
        x = s_long[j];
        c = off[x.x];
        end = off[x.x + 1];
      }
      const uint32_t stop = end - c > PL_GROUP_MAX ? c + PL_GROUP_MAX : end;
      c += 4;
      bool hit = false;  // the group's row is done; it waits for the wave's others
      while (__ballot(c < stop)) {
        int32_t at, got = -1;
        probe_row(col, fbits, c, stop, first, PL_GROUP, &at, &got);
        if (c < stop) {
          hit = at >= 0;
          if (lane == first) {
            const int32_t took = stop - c < 4 * PL_GROUP ? (int32_t)(stop - c) : 4 * PL_GROUP;
            insp += hit ? at + 1 : took;
            if (hit) {
              depth[x.x] = d_new;
              if (parent) parent[x.x] = got;
              atomicOr(&s_new[x.y], 1ull << (x.x & 63));
            }
          }
          c = hit ? stop : c + 4 * PL_GROUP;
        }
      }
      stage.push(hit && lane == first, x.x);
      const bool more = lane == first && !hit && end > stop;
      const uint64_t mask = __ballot(more);
      if (mask) {
        int32_t pos = 0;
        if (lane == 0) pos = atomicAdd(&s_nhub, __popcll(mask));
        pos = __builtin_amdgcn_readfirstlane(pos);
        if (more) s_hub[pos + fg_mbcnt(mask)] = x;
      }
    }
    __syncthreads();
    const int32_t nhub = s_nhub;
    for (int32_t j = wid; j < nhub; j += PL_WAVES) {
      const int2 x = s_hub[j];
      const uint32_t end = off[x.x + 1];
      for (uint32_t c = off[x.x] + PL_GROUP_MAX; c < end; c += 4 * FG_WAVE) {
        int32_t at, got = -1;
        probe_row(col, fbits, c, end, 0, FG_WAVE, &at, &got);
        if (at >= 0) {
          if (lane == 0) {
            insp += at + 1;
            depth[x.x] = d_new;
            if (parent) parent[x.x] = got;
            atomicOr(&s_new[x.y], 1ull << (x.x & 63));
          }
          stage.push(lane == 0, x.x);
          break;
        }
        if (lane == 0) insp += end - c < 4 * FG_WAVE ? (int32_t)(end - c) : 4 * FG_WAVE;
      }
    }
    __syncthreads();
    if (lane == 0 && w < nwords) {
      const uint64_t nb = s_new[wid];
      next_bits[w] = nb;
      if (nb) visited[w] = vis | nb;
    }
    stage.flush_above(PL_STAGE - PL_BT, out_q, out_len);
  }
  stage.flush_above(0, out_q, out_len);
  insp = fg_block_sum<PL_BT>(insp, s_red);
  if (threadIdx.x == 0 && inspected && insp)
    atomicAdd((unsigned long long*)inspected, (unsigned long long)insp);
}

// Clears the pull step's two counters.
__global__ void pull_clear_kernel(int32_t* out_len, int64_t* inspected) {
  if (threadIdx.x == 0) {
    *out_len = 0;
    if (inspected) *inspected = 0;
  }
}

// ---------------------------------------------------------- conversions

__global__ void queue_to_bitmap_kernel(const int32_t* __restrict__ q, int64_t len,
                                       unsigned long long* __restrict__ bits) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t v = q[i];
    atomicOr(&bits[v >> 6], 1ull << (v & 63));
  }
}

// The set bits of QB words per workgroup, at their place in the queue (the
// popcounts scanned here, the tiles before from the tile sums).  A wave
// writes its words one after another, a lane per bit, so the stores of a
// word are contiguous; empty words are skipped.
template <bool SELF>
__global__ void bitmap_to_queue_kernel(int64_t nwords, const uint64_t* __restrict__ bits,
                                       const int64_t* __restrict__ sums,
                                       const int64_t* __restrict__ total,
                                       int32_t* __restrict__ out_q, int32_t* __restrict__ out_len) {
  __shared__ int64_t red[QB / FG_WAVE + 1];
  const int lane = fg_lane();
  const int64_t i = (int64_t)blockIdx.x * QB + threadIdx.x;
  const uint64_t w = i < nwords ? bits[i] : 0ull;
  const int64_t base = tile_base<SELF, QB>(sums, red);
  int64_t tot = 0;
  const int64_t ex = fg_block_excl_scan<QB>((int64_t)__popcll(w), red, &tot);
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
    *out_len = (int32_t)(SELF ? base + tot : *total);
  const int32_t pos = (int32_t)(base + ex);
  uint64_t some = __ballot(w != 0);
  // sparse words: a word per lane, bit after bit, takes as many steps as the
  // fullest word has bits (67 M vertices, a bit in twenty: 46 us word by word,
  // 30 so; half of them set: 48 and 167)
  int32_t most = __popcll(w);
  for (int d = FG_WAVE / 2; d > 0; d >>= 1) {
    const int32_t o = __shfl_xor(most, d, FG_WAVE);
    most = o > most ? o : most;
  }
  if (4 * most < __popcll(some)) {
    int32_t p = pos;
    for (uint64_t x = w; x; x &= x - 1) out_q[p++] = (int32_t)(i * 64 + __builtin_ctzll(x));
    return;
  }
  while (some) {
    const int l = __builtin_ctzll(some);
    some &= some - 1;
    const uint64_t x = fg_readlane64(w, l);
    const int32_t p = __builtin_amdgcn_readlane(pos, l);
    if ((x >> lane) & 1ull) out_q[p + fg_mbcnt(x)] = (int32_t)((i - lane + l) * 64 + lane);
  }
}

// ------------------------------------------------------------- layouts

struct OpsLayout {
  int64_t* sums;
  int64_t* scan;
  int64_t* total;
  int64_t* misc;     // [0] edge-frontier length, [1] inspected
  int32_t* len32;    // [0] out length
  uint32_t* visited; // unfused BFS
  int32_t* q[2];
  int32_t* edst;
  int32_t* esrc;
  size_t bytes;
};

OpsLayout ops_layout(const fg_graph* g, void* ws, bool with_bfs) {
  fg_carver c(ws);
  OpsLayout L;
  const int64_t n = g->n;
  const int64_t maxlen = n > g->nwords ? n : g->nwords;
  L.sums = c.take<int64_t>((maxlen + TB - 1) / TB + 1);
  L.scan = c.take<int64_t>(maxlen + 1);
  L.total = c.take<int64_t>(1);
  L.misc = c.take<int64_t>(4);
  L.len32 = c.take<int32_t>(4);
  if (with_bfs) {
    L.visited = c.take<uint32_t>((n + 31) / 32 + 2);
    L.q[0] = c.take<int32_t>(n);
    L.q[1] = c.take<int32_t>(n);
    L.edst = c.take<int32_t>(g->m > 0 ? g->m : 1);
    L.esrc = c.take<int32_t>(g->m > 0 ? g->m : 1);
  } else {
    L.visited = nullptr;
    L.q[0] = L.q[1] = nullptr;
    L.edst = L.esrc = nullptr;
  }
  L.bytes = c.used;
  return L;
}

int grid_for(int64_t work, int per_block, int cap) {
  int64_t b = (work + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (int)b;
}

}  // namespace

size_t fg_ops_workspace_bytes(const fg_graph* g, bool with_bfs) {
  return ops_layout(g, nullptr, with_bfs).bytes;
}


extern "C" size_t fg_workspace_bytes(const fg_graph* g, int32_t primitive, int32_t lanes) {
  if (!g) return 0;
  switch (primitive) {
    case FG_PRIM_BFS: return fg_bfs_workspace_bytes(g);
    case FG_PRIM_BFS_UNFUSED: return fg_ops_workspace_bytes(g, true);
    case FG_PRIM_SSSP: return fg_sssp_workspace_bytes(g);
    case FG_PRIM_MSBFS:
      if (lanes < 1 || lanes > 64) return 0;
      return fg_msbfs_workspace_bytes(g, lanes);
    case FG_PRIM_MSSSP:
      if (lanes < 1 || lanes > 64) return 0;
      return fg_mssp_workspace_bytes(g);
    case FG_PRIM_PR: return fg_pr_workspace_bytes(g);
    case FG_PRIM_CC: return fg_cc_workspace_bytes(g);
    default: return 0;
  }
}

static fg_status advance_impl(const fg_graph* g, const int32_t* frontier, int64_t len,
                              const int32_t* len_dev, int32_t* out_dst, int32_t* out_src,
                              int64_t capacity, int64_t* out_len, const OpsLayout& L,
                              hipStream_t s) {
  ScanWs sw{L.sums, L.scan, L.total};
  // with a device-resident length the scan runs over the host bound `len`,
  // entries past the device length contributing no edges
  run_scan(len, DegOf{g->off, frontier, len_dev}, sw, s);
  int blocks = grid_for(g->m > 0 ? g->m : 1, EXP_PER_BLOCK, 4096);
  advance_expand_kernel<<<blocks, 256, 0, s>>>(len, frontier, g->off, g->col, L.scan, L.total,
                                               capacity, out_dst, out_src, out_len);
  FG_HIP_TRY(hipGetLastError());
  return FG_OK;
}

extern "C" fg_status fg_advance(const fg_graph* g, const int32_t* frontier, int32_t len,
                                const int32_t* len_dev, int32_t* out_dst, int32_t* out_src,
                                int64_t capacity, int64_t* out_len, void* ws, size_t ws_bytes,
                                void* stream) {
  if (!g || !out_dst || !out_src || !out_len || !ws)
    return fg_set_error(FG_EINVAL, "fg_advance: NULL argument");
  if (len < 0 || len > g->n) return fg_set_error(FG_EINVAL, "fg_advance: len=%d outside [0, n]", len);
  if (len > 0 && !frontier) return fg_set_error(FG_EINVAL, "fg_advance: frontier is NULL");
  if (capacity < 0) return fg_set_error(FG_EINVAL, "fg_advance: negative capacity");
  OpsLayout L = ops_layout(g, ws, false);
  FG_CHECK_WS_ALIGN(ws, "fg_advance");
  if (ws_bytes < L.bytes)
    return fg_set_error(FG_ENOMEM, "fg_advance: workspace of %zu bytes < required %zu", ws_bytes,
                        L.bytes);
  return advance_impl(g, frontier, len, len_dev, out_dst, out_src, capacity, out_len, L,
                      (hipStream_t)stream);
}

extern "C" fg_status fg_filter(const fg_graph* g, const int32_t* dst, const int32_t* src,
                               int64_t len, const int64_t* len_dev, uint32_t* visited,
                               int32_t iter, int32_t* depth, int32_t* parent, int32_t* out_q,
                               int32_t* out_len, void* stream) {
  if (!g || !visited || !depth || !out_q || !out_len)
    return fg_set_error(FG_EINVAL, "fg_filter: NULL argument");
  if (len < 0) return fg_set_error(FG_EINVAL, "fg_filter: negative len");
  if (len > 0 && (!dst || (parent && !src))) return fg_set_error(FG_EINVAL, "fg_filter: NULL edge frontier");
  if (iter < 0) return fg_set_error(FG_EINVAL, "fg_filter: negative iteration");
  hipStream_t s = (hipStream_t)stream;
  fill_i32_kernel<<<1, 64, 0, s>>>(out_len, 1, 0);
  if (len > 0)
    filter_kernel<<<grid_for(len, FT_BT, 512), FT_BT, 0, s>>>(
        dst, src, len_dev, len, len, visited, iter + 1, depth, parent, out_q, out_len);
  FG_HIP_TRY(hipGetLastError());
  return FG_OK;
}

extern "C" fg_status fg_pull_step(const fg_graph* g, const uint64_t* frontier_bits,
                                  uint64_t* visited, uint64_t* next_bits, int32_t iter,
                                  int32_t* depth, int32_t* parent, int32_t* out_q,
                                  int32_t* out_len, int64_t* inspected, void* stream) {
  if (!g || !frontier_bits || !visited || !next_bits || !depth || !out_q || !out_len)
    return fg_set_error(FG_EINVAL, "fg_pull_step: NULL argument");
  if (!g->symmetric)
    return fg_set_error(FG_EUNSUPPORTED, "fg_pull_step: needs an undirected graph (FG_SYMMETRIC)");
  if (iter < 0) return fg_set_error(FG_EINVAL, "fg_pull_step: negative iteration");
  hipStream_t s = (hipStream_t)stream;
  pull_clear_kernel<<<1, 64, 0, s>>>(out_len, inspected);
  pull_step_kernel<<<grid_for(g->nwords, PL_WAVES, PL_GRID), PL_BT, 0, s>>>(
      g->nwords, g->off, g->col, g->head, g->nzmask, (const uint32_t*)frontier_bits, visited,
      next_bits, iter + 1, depth, parent, out_q, out_len, inspected);
  FG_HIP_TRY(hipGetLastError());
  return FG_OK;
}

extern "C" fg_status fg_queue_to_bitmap(const fg_graph* g, const int32_t* queue, int32_t len,
                                        uint64_t* bits, void* stream) {
  if (!g || !bits) return fg_set_error(FG_EINVAL, "fg_queue_to_bitmap: NULL argument");
  if (len < 0 || len > g->n) return fg_set_error(FG_EINVAL, "fg_queue_to_bitmap: bad len %d", len);
  if (len > 0 && !queue) return fg_set_error(FG_EINVAL, "fg_queue_to_bitmap: queue is NULL");
  if (len == 0) return FG_OK;
  queue_to_bitmap_kernel<<<grid_for(len, 256, 4096), 256, 0, (hipStream_t)stream>>>(
      queue, len, (unsigned long long*)bits);
  FG_HIP_TRY(hipGetLastError());
  return FG_OK;
}

extern "C" fg_status fg_bitmap_to_queue(const fg_graph* g, const uint64_t* bits, int32_t* out_q,
                                        int32_t* out_len, void* ws, size_t ws_bytes,
                                        void* stream) {
  if (!g || !bits || !out_q || !out_len || !ws)
    return fg_set_error(FG_EINVAL, "fg_bitmap_to_queue: NULL argument");
  OpsLayout L = ops_layout(g, ws, false);
  FG_CHECK_WS_ALIGN(ws, "fg_bitmap_to_queue");
  if (ws_bytes < L.bytes)
    return fg_set_error(FG_ENOMEM, "fg_bitmap_to_queue: workspace of %zu bytes < required %zu",
                        ws_bytes, L.bytes);
  hipStream_t s = (hipStream_t)stream;
  const unsigned tiles = (unsigned)(((int64_t)g->nwords + QB - 1) / QB);
  tile_sum_kernel<QB><<<tiles, QB, 0, s>>>((int64_t)g->nwords, PopOf{bits}, L.sums);
  if (tiles <= SELF_TILES) {
    bitmap_to_queue_kernel<true><<<tiles, QB, 0, s>>>(g->nwords, bits, L.sums, L.total, out_q,
                                                      out_len);
  } else {
    scan_sums_kernel<<<1, TB, 0, s>>>(tiles, L.sums, L.total);
    bitmap_to_queue_kernel<false><<<tiles, QB, 0, s>>>(g->nwords, bits, L.sums, L.total, out_q,
                                                       out_len);
  }
  FG_HIP_TRY(hipGetLastError());
  return FG_OK;
}

// Unfused push BFS (Alg. 1: an advance kernel followed by a filter kernel),
// driven from the host one iteration at a time.  Kept as the baseline that
// kernel fusion (Sec. VI-C) is measured against.

fg_status fg_bfs_unfused(const fg_graph* g, int32_t src, void* ws, size_t ws_bytes,
                         int32_t* depth, int32_t* parent, fg_run_stats* stats, hipStream_t s) {
  OpsLayout L = ops_layout(g, ws, true);
  FG_CHECK_WS_ALIGN(ws, "fg_bfs_unfused");
  if (ws_bytes < L.bytes)
    return fg_set_error(FG_ENOMEM, "fg_bfs: workspace of %zu bytes < required %zu (unfused)",
                        ws_bytes, L.bytes);
  fg_bfs_launch_init(g, src, depth, parent, (uint64_t*)L.visited, L.q[0], stats, s, nullptr, 0);
  std::vector<int8_t> dir;
  std::vector<int64_t> front, insp;
  int64_t len = 1, reached = 1, insp_sum = 0;
  int32_t k = 0, sel = 0;
  while (len > 0) {
    front.push_back(len);
    fg_status st = advance_impl(g, L.q[sel], len, nullptr, L.edst, L.esrc, g->m, L.misc, L, s);
    if (st != FG_OK) return st;
    fill_i32_kernel<<<1, 64, 0, s>>>(L.len32, 1, 0);
    filter_kernel<<<grid_for(g->m > 0 ? g->m : 1, FT_BT, 512), FT_BT, 0, s>>>(
        L.edst, L.esrc, L.misc, 0, g->m, L.visited, k + 1, depth, parent, L.q[sel ^ 1], L.len32);
    int64_t h[1];
    int32_t nl = 0;
    FG_HIP_TRY(hipMemcpyAsync(h, L.misc, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    FG_HIP_TRY(hipMemcpyAsync(&nl, L.len32, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    FG_HIP_TRY(hipStreamSynchronize(s));
    insp.push_back(h[0]);
    insp_sum += h[0];
    len = nl;
    reached += nl;
    sel ^= 1;
    k++;
  }
  if (stats) {
    fg_run_stats hs;
    memset(&hs, 0, sizeof(hs));
    hs.status = FG_OK;
    hs.iterations = k;
    hs.reached = reached;
    hs.edges_inspected = insp_sum;
    for (int32_t i = 0; i < k && i < FG_TRACE_MAX; ++i) {
      hs.dir[i] = 0;
      hs.frontier[i] = front[i];
      hs.inspected[i] = insp[i];
    }
    FG_HIP_TRY(hipMemcpyAsync(stats, &hs, sizeof(hs), hipMemcpyHostToDevice, s));
    FG_HIP_TRY(hipStreamSynchronize(s));
  }
  return FG_OK;
}
