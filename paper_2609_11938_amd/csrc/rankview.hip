// Launch-order view of launches whose seq is not promised dense: the rank of
// every launch among all seq values, in one pass over memory per step instead
// of a four-pass radix sort of (seq, launch) pairs.
//   1. k_rv_range    smallest and largest seq
//   2. k_rv_count    launches per bucket of equal width over that range
//   3. k_rv_base     exclusive prefix of the counts
//   4. k_rv_scatter  (seq, launch) records to their buckets, in any order
//   5. k_rv_rank     per bucket: a bitmap of its seq values in LDS; a launch's
//                    rank is the bucket's base plus the set bits below its own
//   6. k_rv_sort     returns at once, unless equal values call for it
// Seq values are unique, so the order inside a bucket needs no sort. The
// buckets are at most 2^18 values wide (all of 32 bits in 16384 buckets) and
// hold about a thousand launches each when seq is spread evenly. Uneven seq (a
// far value beside a dense run, two captures far apart) leaves nearly all
// launches in a few buckets: step 3 lists the overfull ones in parts, and in
// step 5 a block per part builds the bucket's bitmap and ranks its part.
// Equal seq values (an error, reported as ORDER) are seen in step 5 as a bit
// already set. A bucket of up to 4096 launches then counts the smaller (seq,
// launch) records for each; after a larger one step 6 sorts all pairs. Either
// way ties go by input index, as the general sort has it. 2M shuffled launches,
// the call: spread evenly 698 us, one far value 707, one pair of equal ones too
// 998 (one block sorted all pairs in 20 ms), all equal 484.
// 3M launches of 8 streams: 77 us (10 + 16 + 7 + 21 + 19 + 4), bound by the
// scatter's partial lines and by the latency of short kernels; the whole call
// 559 us with the sort, 375 us with this. 500k shuffled: 328 us and 229 us.
// Blocks of 256 and 1024 threads in step 5 and 2048 launches per bucket: the
// same within 3 us. Eight loads in flight there, or a loop of its own for the
// parts: 4M launches 7 us longer, the call (beside its other streams' kernels).
#include "common.h"
#include "impl.h"

namespace opa {

constexpr int kRvThreads = 1024, kRvPer = 8, kRvTile = kRvThreads * kRvPer;
constexpr int kRvPerBits = 10;  // log2 of the launches wanted per bucket
constexpr int kRvWords = (1 << kRvWidthBits) / 32;

struct RvArgs {
  const uint32_t *seq;
  int64_t T;
  // [0] smallest, [1] largest seq, [2] parts of overfull buckets, [3] equal
  // values in a large bucket, [4] next work item of k_rv_sort, [8 + p] items
  // of its phase p that are done
  uint32_t *mm;
  uint32_t *cnt, *cur; // [kRvBuckets + 1] counts, then bases; next free place
  uint64_t *rec;       // [T] seq << 32 | launch, by bucket
  int32_t *sv, *rk;
  opattr_diag *diag;
  uint32_t *k0, *k1, *v0, *v1;  // [T] each: the sort of k_rv_sort (rec is k0 and k1)
  uint32_t *hist;               // [kRvItems][256] digit counts of the sort's items
  uint2 *part;                  // parts of overfull buckets: bucket, first launch in it
};

// Launches of a bucket from which it is ranked in parts, and of a part. By one
// block a bucket, 2M launches in 256 buckets of 7,812 took 71 us longer, in 8
// buckets 720 us longer than spread evenly; in parts 0 and 7 us longer. Up to
// 4096 launches are two rounds of a block's loads.
constexpr uint32_t kRvFull = 4096, kRvPart = 8192;
__host__ __device__ inline uint32_t rv_full(int64_t T) {  // (even buckets of long lists hold more)
  const int64_t even = 4 * (T / kRvBuckets);
  return even > kRvFull ? (uint32_t)even : kRvFull;
}
// (a bucket of n > kRvFull launches has at most 2 n / kRvPart parts)
inline size_t rv_max_parts(int64_t T) { return (size_t)(2 * T / kRvPart + 1); }

// log2 of the buckets' width: about T >> per_bits buckets over the range, but
// none wider than the bitmap
__device__ __forceinline__ int rv_shift(const RvArgs &a, uint32_t lo, uint32_t hi) {
  const uint32_t range = hi - lo;
  const int rb = bits_for(range);
  int nb = 0;  // log2 of the buckets wanted
  while (((int64_t)1 << (kRvPerBits + nb)) < a.T) ++nb;
  int s = rb - nb;
  s = s < 0 ? 0 : s;
  s = s > kRvWidthBits ? kRvWidthBits : s;
  const int least = 32 - kRvWidthBits;  // log2(kRvBuckets)
  return rb - s > least ? rb - least : s;
}

__global__ void __launch_bounds__(kRvThreads) k_rv_range(RvArgs a) {
  __shared__ uint32_t red[2][kRvThreads / OPA_WAVE];
  uint32_t lo = 0xFFFFFFFFu, hi = 0;
  for (int64_t i0 = (int64_t)blockIdx.x * kRvTile + threadIdx.x; i0 < a.T;
       i0 += (int64_t)gridDim.x * kRvTile) {
    uint32_t v[kRvPer];
#pragma unroll
    for (int k = 0; k < kRvPer; ++k) {  // past the end: the last one once more
      const int64_t i = i0 + k * kRvThreads;
      v[k] = a.seq[i < a.T ? i : a.T - 1];
    }
#pragma unroll
    for (int k = 0; k < kRvPer; ++k) {
      lo = v[k] < lo ? v[k] : lo;
      hi = v[k] > hi ? v[k] : hi;
    }
  }
#pragma unroll
  for (int o = OPA_WAVE / 2; o > 0; o >>= 1) {
    const uint32_t x = __shfl_xor(lo, o, OPA_WAVE), y = __shfl_xor(hi, o, OPA_WAVE);
    lo = x < lo ? x : lo;
    hi = y > hi ? y : hi;
  }
  if (lane_id() == 0) {
    red[0][wave_id()] = lo;
    red[1][wave_id()] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kRvThreads / OPA_WAVE; ++w) {
      lo = red[0][w] < lo ? red[0][w] : lo;
      hi = red[1][w] > hi ? red[1][w] : hi;
    }
    atomicMin(&a.mm[0], lo);
    atomicMax(&a.mm[1], hi);
  }
}

// bucket counts of a tile in LDS; the thread's seq values and their places
// among the tile's launches of the bucket
__device__ __forceinline__ void rv_tile(const RvArgs &a, int shift, uint32_t lo, uint32_t nb,
                                        uint32_t *l, uint32_t (&s)[kRvPer], uint32_t (&p)[kRvPer]) {
  for (uint32_t x = threadIdx.x; x < nb; x += kRvThreads) l[x] = 0;
  const int64_t base = (int64_t)blockIdx.x * kRvTile;
#pragma unroll
  for (int k = 0; k < kRvPer; ++k) {
    const int64_t i = base + k * kRvThreads + threadIdx.x;
    s[k] = i < a.T ? a.seq[i] : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kRvPer; ++k) {
    const int64_t i = base + k * kRvThreads + threadIdx.x;
    if (i < a.T) p[k] = atomicAdd(&l[(s[k] - lo) >> shift], 1u);
  }
  __syncthreads();
}

__global__ void __launch_bounds__(kRvThreads) k_rv_count(RvArgs a) {
  extern __shared__ __align__(16) unsigned char rv_raw[];
  uint32_t *l = reinterpret_cast<uint32_t *>(rv_raw);
  const uint32_t lo = a.mm[0], hi = a.mm[1];
  const int shift = rv_shift(a, lo, hi);
  const uint32_t nb = ((hi - lo) >> shift) + 1u;
  uint32_t s[kRvPer], p[kRvPer];
  rv_tile(a, shift, lo, nb, l, s, p);
  for (uint32_t x = threadIdx.x; x < nb; x += kRvThreads)
    if (l[x]) atomicAdd(&a.cnt[x], l[x]);
}

__global__ void __launch_bounds__(1024) k_rv_base(RvArgs a) {
  __shared__ uint32_t sh[16];
  constexpr int kQuads = kRvBuckets / 1024 / 4;
  uint4 v[kQuads];
  uint4 *cnt = reinterpret_cast<uint4 *>(a.cnt) + threadIdx.x * kQuads;
  uint4 *cur = reinterpret_cast<uint4 *>(a.cur) + threadIdx.x * kQuads;
  uint32_t sum = 0;
#pragma unroll
  for (int k = 0; k < kQuads; ++k) v[k] = cnt[k];
#pragma unroll
  for (int k = 0; k < kQuads; ++k) sum += v[k].x + v[k].y + v[k].z + v[k].w;
  uint32_t run = block_excl_scan_add<uint32_t>(sum, sh, nullptr);
#pragma unroll
  for (int k = 0; k < kQuads; ++k) {
    const uint4 e = make_uint4(run, run + v[k].x, run + v[k].x + v[k].y,
                               run + v[k].x + v[k].y + v[k].z);
    run = e.w + v[k].w;
    cnt[k] = e;
    cur[k] = e;
  }
  if (threadIdx.x == 1023) a.cnt[kRvBuckets] = run;
  // the overfull buckets' parts
  const uint32_t full = rv_full(a.T);
  auto parts = [&](uint32_t n) { return n > full ? (n + kRvPart - 1) / kRvPart : 0u; };
  uint32_t np = 0, total;
#pragma unroll
  for (int k = 0; k < kQuads; ++k) np += parts(v[k].x) + parts(v[k].y) + parts(v[k].z) + parts(v[k].w);
  if (!__syncthreads_or(np != 0)) return;
  uint32_t p = block_excl_scan_add<uint32_t>(np, sh, &total);
  if (threadIdx.x == 0) a.mm[2] = total;
  if (np == 0) return;
  const uint32_t b0 = threadIdx.x * 4 * kQuads, b1 = b0 + 4 * kQuads;
  for (uint32_t b = b0; b < b1; ++b) {  // (the counts are bases by now; run: the end of the last)
    const uint32_t n = (b + 1 < b1 ? a.cnt[b + 1] : run) - a.cnt[b];
    for (uint32_t q = 0; q < parts(n); ++q) a.part[p++] = make_uint2(b, q * kRvPart);
  }
}

__global__ void __launch_bounds__(kRvThreads) k_rv_scatter(RvArgs a) {
  extern __shared__ __align__(16) unsigned char rv_raw[];
  uint32_t *l = reinterpret_cast<uint32_t *>(rv_raw);
  const uint32_t lo = a.mm[0], hi = a.mm[1];
  const int shift = rv_shift(a, lo, hi);
  const uint32_t nb = ((hi - lo) >> shift) + 1u;
  uint32_t s[kRvPer], p[kRvPer];
  rv_tile(a, shift, lo, nb, l, s, p);
  for (uint32_t x = threadIdx.x; x < nb; x += kRvThreads)
    if (l[x]) l[x] = atomicAdd(&a.cur[x], l[x]);
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kRvTile;
#pragma unroll
  for (int k = 0; k < kRvPer; ++k) {
    const int64_t i = base + k * kRvThreads + threadIdx.x;
    if (i < a.T) a.rec[l[(s[k] - lo) >> shift] + p[k]] = ((uint64_t)s[k] << 32) | (uint32_t)i;
  }
}

constexpr int kRvRankThreads = 512, kRvUnroll = 4;
constexpr uint32_t kRvEqualMax = 4096;

struct RvRankLds {
  uint32_t bits[kRvWords];
  uint32_t tb[kRvRankThreads];  // set bits before each thread's words
  uint32_t sh[kRvRankThreads / OPA_WAVE];
};

// The launches [i_lo, i_hi) of bucket b (places inside it) ranked, by the
// whole block. kRvUnroll of a thread's records are in flight while the bitmap of
// the whole bucket is built.
__device__ __forceinline__ void rv_rank_bucket(const RvArgs &a, int shift, uint32_t lo, uint32_t b,
                                               uint32_t i_lo, uint32_t i_hi, RvRankLds &l) {
  const int tid = threadIdx.x;
  const uint32_t words = shift > 5 ? 1u << (shift - 5) : 1u, mask = (1u << shift) - 1u;
  const uint32_t ch = (words + kRvRankThreads - 1) / kRvRankThreads;
  const uint32_t x0 = a.cnt[b], n = a.cnt[b + 1] - x0;
  if (i_hi > n) i_hi = n;
  const uint64_t *rec = a.rec + x0;
  const uint32_t *val = reinterpret_cast<const uint32_t *>(rec) + 1;  // every other word
  uint32_t set = 0;
  if (n <= 1u << shift) {  // else there are equal values
    for (uint32_t x = tid; x < words; x += kRvRankThreads) l.bits[x] = 0;
    __syncthreads();
    for (uint32_t i0 = tid; i0 < n; i0 += kRvRankThreads * kRvUnroll) {
      uint32_t v[kRvUnroll];
#pragma unroll
      for (int k = 0; k < kRvUnroll; ++k) {
        const uint32_t i = i0 + k * kRvRankThreads;
        v[k] = (val[2 * (size_t)(i < n ? i : i0)] - lo) & mask;  // past the end: the first once more
      }
#pragma unroll
      for (int k = 0; k < kRvUnroll; ++k)
        if (i0 + k * kRvRankThreads < n) atomicOr(&l.bits[v[k] >> 5], 1u << (v[k] & 31));
    }
    __syncthreads();
    uint32_t c = 0;
    for (uint32_t k = 0; k < ch; ++k) {
      const uint32_t x = tid * ch + k;
      if (x < words) c += (uint32_t)__popc(l.bits[x]);
    }
    l.tb[tid] = x0 + block_excl_scan_add<uint32_t>(c, l.sh, &set);
    __syncthreads();
  }
  if (set != n) {  // equal values; uniform
    if (tid == 0) {
      if (n > kRvEqualMax) a.mm[3] = 1u;
      atomicOr(&a.diag->flags, OPATTR_F_ORDER);
    }
    if (n <= kRvEqualMax)
      for (uint32_t i = tid; i < n; i += kRvRankThreads) {
        const uint64_t r = rec[i];
        uint32_t q = x0;
        for (uint32_t j = 0; j < n; ++j) q += rec[j] < r ? 1u : 0u;
        a.sv[q] = (int32_t)(uint32_t)r;
        a.rk[(uint32_t)r] = (int32_t)q;
      }
  } else {
    for (uint32_t i0 = i_lo + tid; i0 < i_hi; i0 += kRvRankThreads * kRvUnroll) {
      uint64_t r[kRvUnroll];
#pragma unroll
      for (int k = 0; k < kRvUnroll; ++k) {
        const uint32_t i = i0 + k * kRvRankThreads;
        r[k] = i < i_hi ? rec[i] : 0u;
      }
#pragma unroll
      for (int k = 0; k < kRvUnroll; ++k) {
        if (i0 + k * kRvRankThreads >= i_hi) continue;
        const uint32_t v = ((uint32_t)(r[k] >> 32) - lo) & mask, wd = v >> 5;
        uint32_t q = l.tb[wd / ch] + (uint32_t)__popc(l.bits[wd] & ((1u << (v & 31)) - 1u));
        for (uint32_t x = wd / ch * ch; x < wd; ++x) q += (uint32_t)__popc(l.bits[x]);
        a.sv[q] = (int32_t)(uint32_t)r[k];
        a.rk[(uint32_t)r[k]] = (int32_t)q;
      }
    }
  }
  __syncthreads();  // the bitmap is free for the next bucket
}

__global__ void __launch_bounds__(kRvRankThreads) k_rv_rank(RvArgs a) {
  __shared__ RvRankLds lds;
  const uint32_t lo = a.mm[0], hi = a.mm[1], np = a.mm[2], full = rv_full(a.T);
  const int shift = rv_shift(a, lo, hi);
  const uint32_t nb = ((hi - lo) >> shift) + 1u;
  for (uint32_t w = blockIdx.x; w < np + nb; w += gridDim.x) {  // parts, then whole buckets
    uint32_t b = w - np, i_lo = 0, i_hi;
    if (w < np) {
      const uint2 e = a.part[w];
      b = e.x;
      i_lo = e.y;
      i_hi = e.y + kRvPart;
    } else {
      i_hi = a.cnt[b + 1] - a.cnt[b];
      if (i_hi == 0 || i_hi > full) continue;  // uniform over the block
    }
    rv_rank_bucket(a, shift, lo, b, i_lo, i_hi, lds);
  }
}

// The sort of all (seq, launch) pairs, only when an earlier step asked for it:
// a stable LSD radix sort of the range's bits, 8 a pass, in one launch. A pass
// is two phases over stretches of tiles, at most kRvItems of them: the
// stretches' digit counts, then the scatter, which adds up the counts before
// its stretch itself; the last one writes the view. The stretches are handed
// out in order by one counter, and before its stretch a block waits for the
// whole phase before: all of that was handed out earlier, to blocks that run
// and wait for still earlier phases only, so every wait ends, however few
// blocks run at a time. (Few stretches, because a stretch ends with the
// write-back of an L2.)
constexpr int kRvSortPer = 4, kRvSortTile = kRvSortPer * kRvThreads;
constexpr int kRvItems = 128, kRvPhases = 8;
constexpr int kRvWaves = kRvThreads / OPA_WAVE;

struct RvSortLds {
  uint16_t cnt[kRvSortPer * kRvWaves * 256];
  uint32_t c[256], part[4][256], less[4][256];
  uint32_t sh[kRvWaves], item;
};

// digit counts of the tiles [t0, t1) to hist[256]
__device__ __forceinline__ void rv_sort_count(const uint32_t *keys, uint32_t lo, int64_t T,
                                              int64_t t0, int64_t t1, int shift, uint32_t *hist,
                                              RvSortLds &l) {
  const int tid = threadIdx.x;
  if (tid < 256) l.c[tid] = 0;
  __syncthreads();
  const int64_t x1 = t1 * kRvSortTile < T ? t1 * kRvSortTile : T;
  for (int64_t x0 = t0 * kRvSortTile + tid; x0 < x1; x0 += kRvSortTile) {
#pragma unroll
    for (int k = 0; k < kRvSortPer; ++k) {
      const int64_t x = x0 + k * kRvThreads;
      if (x < x1) atomicAdd(&l.c[((keys[x] - lo) >> shift) & 255u], 1u);
    }
  }
  __syncthreads();
  if (tid < 256) hist[tid] = l.c[tid];
}

// The tiles [t0, t1) of item k (of n items, hist their counts) scattered; with
// out.sv the places are the launches' ranks.
struct RvOut {
  uint32_t *key, *val;
  int32_t *sv, *rk;
};
__device__ __forceinline__ void rv_sort_scatter(const uint32_t *ki, const uint32_t *vi,
                                                const RvOut &out, uint32_t lo, int64_t T,
                                                int64_t t0, int64_t t1, int shift,
                                                const uint32_t *hist, uint32_t k, uint32_t n,
                                                RvSortLds &l) {
  const int tid = threadIdx.x, w = wave_id();
  {  // each digit's launches in all items, and in those before k: four threads a digit
    const int d = tid & 255, q = tid >> 8;
    uint32_t all = 0, less = 0;
#pragma unroll 8
    for (uint32_t x = q; x < n; x += 4) {
      const uint32_t v = hist[x * 256 + d];
      all += v;
      less += x < k ? v : 0u;
    }
    l.part[q][d] = all;
    l.less[q][d] = less;
    __syncthreads();
    uint32_t v = 0, b = 0;
    if (tid < 256)
      for (int y = 0; y < 4; ++y) {
        v += l.part[y][tid];
        b += l.less[y][tid];
      }
    const uint32_t e = block_excl_scan_add<uint32_t>(v, l.sh, nullptr);
    if (tid < 256) l.c[tid] = e + b;  // the digit's next place
  }
  uint32_t *c32 = reinterpret_cast<uint32_t *>(l.cnt);
  for (int64_t t = t0; t < t1; ++t) {
    for (int x = tid; x < kRvSortPer * kRvWaves * 256 / 2; x += kRvThreads) c32[x] = 0;
    __syncthreads();
    uint32_t key[kRvSortPer], val[kRvSortPer], lr[kRvSortPer];
#pragma unroll
    for (int j = 0; j < kRvSortPer; ++j) {
      const int64_t x = t * kRvSortTile + j * kRvThreads + tid;
      const bool ok = x < T;
      key[j] = ok ? ki[x] : lo;
      val[j] = ok ? (vi ? vi[x] : (uint32_t)x) : 0u;
    }
#pragma unroll
    for (int j = 0; j < kRvSortPer; ++j) {
      const bool ok = t * kRvSortTile + j * kRvThreads + tid < T;
      const uint32_t d = ((key[j] - lo) >> shift) & 255u;
      const uint64_t pm = peers8(d) & __ballot(ok);
      lr[j] = (uint32_t)__popcll(pm & lanemask_lt());
      if (ok && lr[j] == 0) l.cnt[(j * kRvWaves + w) * 256 + d] = (uint16_t)__popcll(pm);
    }
    __syncthreads();
    {  // the digit's counts over (j, wave), in order: four threads a digit again
      constexpr int kQ = kRvSortPer * kRvWaves / 4;
      const int d = tid & 255, q = tid >> 8;
      uint32_t v[kQ], run = 0;
#pragma unroll
      for (int y = 0; y < kQ; ++y) {
        v[y] = l.cnt[(q * kQ + y) * 256 + d];
        run += v[y];
      }
      l.part[q][d] = run;
      if (q == 0) l.less[0][d] = l.c[d];  // the digit's first place in this tile
      __syncthreads();
      run = 0;
      for (int y = 0; y < q; ++y) run += l.part[y][d];
#pragma unroll
      for (int y = 0; y < kQ; ++y) {
        l.cnt[(q * kQ + y) * 256 + d] = (uint16_t)run;
        run += v[y];
      }
      if (q == 3) l.c[d] = l.less[0][d] + run;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kRvSortPer; ++j) {
      if (t * kRvSortTile + j * kRvThreads + tid >= T) continue;
      const uint32_t d = ((key[j] - lo) >> shift) & 255u;
      const uint32_t dst = l.less[0][d] + l.cnt[(j * kRvWaves + w) * 256 + d] + lr[j];
      if (out.sv) {
        out.sv[dst] = (int32_t)val[j];
        out.rk[val[j]] = (int32_t)dst;
      } else {
        out.key[dst] = key[j];
        out.val[dst] = val[j];
      }
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kRvThreads) k_rv_sort(RvArgs a) {
  if (a.mm[3] == 0) return;  // uniform: written by earlier kernels only
  __shared__ RvSortLds l;
  const int tid = threadIdx.x;
  const uint32_t lo = a.mm[0];
  const int64_t nt = (a.T + kRvSortTile - 1) / kRvSortTile;
  const uint32_t n = nt < kRvItems ? (uint32_t)nt : (uint32_t)kRvItems;  // items of a phase
  const uint32_t passes = ((uint32_t)bits_for(a.mm[1] - lo) + 7) / 8;
  for (;;) {
    __syncthreads();
    if (tid == 0) l.item = atomicAdd(&a.mm[4], 1u);
    __syncthreads();
    const uint32_t phase = l.item / n, k = l.item - phase * n, pass = phase >> 1;
    if (pass >= passes) return;  // uniform
    if (phase > 0) {
      if (tid == 0) {
        while (__hip_atomic_load(&a.mm[8 + phase - 1], __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT) < n)
          __builtin_amdgcn_s_sleep(2);
        __threadfence();
      }
      __syncthreads();
    }
    const int64_t t0 = nt * k / n, t1 = nt * (k + 1) / n;
    const int shift = 8 * (int)pass;
    const bool odd = pass & 1u, last = pass + 1 == passes;
    const uint32_t *ki = pass == 0 ? a.seq : odd ? a.k0 : a.k1;
    const uint32_t *vi = pass == 0 ? nullptr : odd ? a.v0 : a.v1;
    if ((phase & 1u) == 0) {
      rv_sort_count(ki, lo, a.T, t0, t1, shift, a.hist + k * 256, l);
    } else {
      const RvOut out{odd ? a.k1 : a.k0, odd ? a.v1 : a.v0, last ? a.sv : nullptr, a.rk};
      rv_sort_scatter(ki, vi, out, lo, a.T, t0, t1, shift, a.hist, k, n, l);
    }
    // the block's writes are made visible before the item counts as done
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) {
      __threadfence();
      __hip_atomic_fetch_add(&a.mm[8 + phase], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

static_assert(8 + kRvPhases <= 64, "the phases' counts");

// the counters and buckets, the sort's digit counts, the overfull buckets' parts
size_t rank_view_entries(int64_t T) {
  return 2 * ((size_t)kRvBuckets + 64) + 64 + kRvItems * 256 + 2 * rv_max_parts(T);
}

void run_rank_view(const opattr_kernels *k, void *ws, const Plan &pl, opattr_diag *diag,
                   hipStream_t s) {
  RvArgs a{};
  a.seq = k->seq;
  a.T = pl.T;
  a.k0 = at<uint32_t>(ws, pl.seqsort_k0);
  a.k1 = at<uint32_t>(ws, pl.seqsort_k1);
  a.v0 = at<uint32_t>(ws, pl.seqsort_v0);
  a.v1 = at<uint32_t>(ws, pl.seqsort_v1);
  a.rec = reinterpret_cast<uint64_t *>(a.k0);  // k0 and k1 are neighbours
  uint32_t *m = at<uint32_t>(ws, pl.rv);
  a.mm = m;
  a.cnt = m + 64;
  a.cur = a.cnt + kRvBuckets + 64;
  a.hist = a.cur + kRvBuckets + 64;
  a.part = reinterpret_cast<uint2 *>(a.hist + kRvItems * 256);
  a.sv = at<int32_t>(ws, pl.sv);
  a.rk = at<int32_t>(ws, pl.rk);
  a.diag = diag;
  FillJobs f;
  f.add(a.mm, 0xFFFFFFFFu, 1);
  f.add(a.mm + 1, 0u, 63 + kRvBuckets + 1);
  fill_many(f, s);
  const unsigned nt = (unsigned)((pl.T + kRvTile - 1) / kRvTile);
  k_rv_range<<<nt < 256 ? nt : 256, kRvThreads, 0, s>>>(a);
  const size_t lds = (size_t)kRvBuckets * 4;
  k_rv_count<<<nt, kRvThreads, lds, s>>>(a);
  k_rv_base<<<1, 1024, 0, s>>>(a);
  k_rv_scatter<<<nt, kRvThreads, lds, s>>>(a);
  const int64_t want = pl.T >> kRvPerBits;
  k_rv_rank<<<(unsigned)(want < 512 ? 512 : (want < kRvBuckets ? want : kRvBuckets)),
              kRvRankThreads, 0, s>>>(a);
  k_rv_sort<<<kRvItems, kRvThreads, 0, s>>>(a);
}

}  // namespace opa
