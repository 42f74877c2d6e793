// Device code of the range stage shared by its own kernels and the compact
// path's multi-job kernels.
#pragma once
#include "common.h"
#include "impl.h"

namespace opa {

constexpr uint64_t kEndLimit = 1ull << 63;  // valid ends stay below 2^63

// validity and effective end of range x (-1 marks a bad range); parents unknown
__device__ __forceinline__ bool rprep_one(const CoreRanges &cr, uint32_t NS, uint32_t NOPS,
                                          int64_t *ree, int32_t *npg, int64_t x) {
  const uint64_t s = cr.s[x], e = cr.e[x];
  const bool ok = cr.st[x] < NS && cr.op[x] < NOPS && s <= e && e < kEndLimit &&
                  (!cr.kind || cr.kind[x] <= OPATTR_KIND_SKIP);
  ree[x] = ok ? (int64_t)e : -1;
  npg[x] = -1;
  return !ok;
}

__device__ __forceinline__ void count_bad(bool bad, opattr_diag *diag) {
  const uint64_t m = __ballot(bad);
  if (m && lane_id() == __ffsll((unsigned long long)m) - 1)
    atomicAdd((unsigned long long *)&diag->bad_records, (unsigned long long)__popcll(m));
}

// tbase[s] = first tile of stream s (tiles never straddle streams), by one
// block
__device__ inline void tile_bases(const int64_t *rblk, uint32_t NS, int32_t *tbase) {
  __shared__ uint32_t sh[16];
  uint32_t carry = 0;
  for (uint32_t base = 0; base < NS; base += blockDim.x) {
    const uint32_t s = base + threadIdx.x;
    uint32_t c = 0;
    // (a broken order promise can leave blocks that overlap or run backwards)
    if (s < NS && rblk[s + 1] > rblk[s])
      c = (uint32_t)((rblk[s + 1] - rblk[s] + kRangeTile - 1) / kRangeTile);
    uint32_t tot;
    const uint32_t pre = block_excl_scan_add<uint32_t>(c, sh, &tot);
    if (s < NS) tbase[s] = (int32_t)(carry + pre);
    carry += tot;
  }
  if (threadIdx.x == 0) tbase[NS] = (int32_t)carry;
}

constexpr uint32_t kInlineBases = 1024;  // streams whose tile bases the tiles find themselves

__device__ __forceinline__ uint32_t stream_of_tile(const int32_t *tbase, uint32_t NS, int32_t t) {
  uint32_t lo = 0, hi = NS;  // last s with tbase[s] <= t
  while (lo + 1 < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (tbase[mid] <= t) lo = mid;
    else hi = mid;
  }
  return lo;
}

struct RangeWork {
  CoreRanges cr;
  uint32_t NS;
  const int64_t *rblk;
  int32_t *tbase;  // written by k_rtile_base, or by the tiles' pass with inline_bases
  int64_t *ree;
  int32_t *npg;
  int64_t *mxv;
  int64_t *tM;
  int32_t *tnpg, *tnpg2;
  int64_t *tmx, *tmx2;
  int32_t *tstr, *tlast;
  uint8_t *sflag;
  opattr_diag *diag;
  int32_t ntr_max;   // tiles there is room for (all of them when the order promise holds)
  int inline_bases;  // the tiles' pass finds the tile bases (NS <= kInlineBases)
};


// (ranges.hip)
RangeWork range_work(const CoreRanges &cr, const opattr_dims *d, void *ws, const Plan &pl,
                     opattr_diag *diag);

// A maximum tree in LDS over kRangeTile values: leaf i at t[kRangeTile + i],
// node n covers the leaves of 2n and 2n + 1. Finding a nearest previous
// greater-or-equal value in it takes at most 2 log2(kRangeTile) LDS reads,
// against one block-wide round per doubling of the longest sibling run for
// pointer jumping (1024 ranges a block: 14 us of rounds, 7 us with the tree).
constexpr int kTreeNodes = 2 * kRangeTile;

// the inner nodes from the leaves; called by the whole block, ends with a barrier
__device__ inline void tree_build(int64_t *t) {
  for (int n = kRangeTile / 2; n >= 1; n >>= 1) {
    __syncthreads();
    for (int k = n + (int)threadIdx.x; k < 2 * n; k += blockDim.x) {
      const int64_t a = t[2 * k], b = t[2 * k + 1];
      t[k] = a > b ? a : b;
    }
  }
  __syncthreads();
}

// the last leaf before leaf i whose value is at least x (-1: none); mx grows
// to the largest value passed on the way to it
__device__ __forceinline__ int tree_prev_ge(const int64_t *t, int i, int64_t x, int64_t &mx) {
  int n = kRangeTile + i;
  bool found = false;
  while (n > 1) {
    if (n & 1) {
      const int64_t v = t[n - 1];
      if (v >= x) {
        --n;
        found = true;
        break;
      }
      mx = v > mx ? v : mx;
    }
    n >>= 1;
  }
  if (!found) return -1;
  while (n < kRangeTile) {
    const int64_t r = t[2 * n + 1];
    if (r >= x) {
      n = 2 * n + 1;
    } else {
      mx = r > mx ? r : mx;
      n = 2 * n;
    }
  }
  return n - kRangeTile;
}

// the largest value of the leaves [lo, hi), at least -1
__device__ __forceinline__ int64_t tree_max(const int64_t *t, int lo, int hi) {
  int64_t m = -1;
  for (int a = lo + kRangeTile, b = hi + kRangeTile; a < b; a >>= 1, b >>= 1) {
    if (a & 1) {
      m = t[a] > m ? t[a] : m;
      ++a;
    }
    if (b & 1) {
      --b;
      m = t[b] > m ? t[b] : m;
    }
  }
  return m;
}

// Local parents inside tile t of kRangeTile ranges: the nearest earlier range
// of the tile whose end is not before the range's (-2: it lies before the
// tile), and the largest end between the two; a skipped end beyond the
// range's start is a crossing. Blocks of kRlThreads.
constexpr int kRlThreads = kRangeTile;
__device__ inline void rlocal_tile(const RangeWork &w, int32_t t, int64_t *tree, int32_t *stb) {
  constexpr int kPer = kRangeTile / kRlThreads;
  const int32_t *tb = w.tbase;
  if (w.inline_bases) {
    tile_bases(w.rblk, w.NS, stb);
    __syncthreads();
    if (t == 0)
      for (uint32_t k = threadIdx.x; k <= w.NS; k += blockDim.x) w.tbase[k] = stb[k];
    tb = stb;
  }
  if (t >= tb[w.NS]) return;  // uniform over the block
  const uint32_t s = stream_of_tile(tb, w.NS, t);
  const int64_t x0 = w.rblk[s] + (int64_t)(t - tb[s]) * kRangeTile;
  const int64_t x1 = min(x0 + kRangeTile, w.rblk[s + 1]);
  int64_t e[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int i = (int)threadIdx.x + u * kRlThreads;
    e[u] = x0 + i < x1 ? w.ree[x0 + i] : -1;
    tree[kRangeTile + i] = e[u];
  }
  tree_build(tree);
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int i = (int)threadIdx.x + u * kRlThreads;
    const int64_t x = x0 + i;
    if (x >= x1) continue;
    int64_t mx = -1;
    const int c = tree_prev_ge(tree, i, e[u], mx);
    w.npg[x] = c >= 0 ? (int32_t)(x0 + c) : -2;
    w.mxv[x] = mx;
    if (c >= 0 && e[u] >= 0 && mx > (int64_t)w.cr.s[x]) w.sflag[s] = 1;
  }
  if (threadIdx.x == 0) {
    w.tM[t] = tree[1];
    w.tstr[t] = (int32_t)s;
    w.tlast[t] = (int32_t)(x1 - 1);
  }
}

// Parent of range x when it lies in an earlier tile u (its maximum end
// reaches x's): down the local parents of that tile from its last range.
// acc holds the largest end between the tiles' and x.
__device__ __forceinline__ void rresolve_in_tile(const RangeWork &w, int64_t x, uint32_t s,
                                                 int64_t ex, int32_t u, int64_t acc) {
  int32_t par = -1;
  if (u >= 0) {
    int32_t y = w.tlast[u];
    int steps = 0;
    while (w.ree[y] < ex && steps < (1 << 20)) {
      const int64_t v = w.ree[y] > w.mxv[y] ? w.ree[y] : w.mxv[y];
      acc = v > acc ? v : acc;
      y = w.npg[y];
      ++steps;
      if (y < 0) break;  // defensive: cannot happen, a tile maximum stops the walk
    }
    par = y;
  }
  w.npg[x] = par;
  if (ex >= 0 && acc > (int64_t)w.cr.s[x]) w.sflag[s] = 1;
}

// The tile that holds range x of stream s (its stream's first tile in t0), or
// -1. Under a broken order promise a stream's block holds ranges of other
// streams, of ids past the last among them, whose tile may not exist.
__device__ __forceinline__ int32_t tile_of_range(const RangeWork &w, uint32_t s, int64_t x,
                                                 int32_t &t0) {
  if (s >= w.NS || x < w.rblk[s] || x >= w.rblk[s + 1]) return -1;
  t0 = w.tbase[s];
  const int32_t t = t0 + (int32_t)((x - w.rblk[s]) / kRangeTile);
  return t < w.ntr_max ? t : -1;
}

// Parents in earlier tiles for the ranges [x0, x0 + blockDim.x), with the
// maximum tree over all tiles (at most kRangeTile of them) built in the
// block: no pass over the tiles of its own.
__device__ inline void rresolve_tree(const RangeWork &w, int64_t x0, int64_t *tree) {
  const int64_t x = x0 + threadIdx.x;
  const bool need = x < w.cr.n && w.npg[x] == -2;
  if (!__syncthreads_or(need)) return;
  const int32_t nt = w.tbase[w.NS], ntr = nt < w.ntr_max ? nt : w.ntr_max;
  for (int k = threadIdx.x; k < kRangeTile; k += blockDim.x)
    tree[kRangeTile + k] = k < ntr ? w.tM[k] : -1;
  tree_build(tree);
  if (!need) return;
  const uint32_t s = w.cr.st[x];
  const int64_t ex = w.ree[x];
  int32_t t0 = 0;
  const int32_t t = tile_of_range(w, s, x, t0);
  if (t < 0) {
    w.npg[x] = -1;
    return;
  }
  int64_t acc = w.mxv[x], skipped = -1;
  int32_t u = tree_prev_ge(tree, t, ex, skipped);
  if (u < t0) {  // none in the stream
    u = -1;
    skipped = tree_max(tree, t0, t);
  }
  acc = skipped > acc ? skipped : acc;
  rresolve_in_tile(w, x, s, ex, u, acc);
}

}  // namespace opa
