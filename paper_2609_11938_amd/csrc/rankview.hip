// Launch-order view of launches whose seq is not promised dense: the rank of
// every launch among all seq values, in one pass over memory per step instead
// of a four-pass radix sort of (seq, launch) pairs.
//   1. k_rv_range    smallest and largest seq
//   2. k_rv_count    launches per bucket of equal width over that range
//   3. k_rv_base     exclusive prefix of the counts
//   4. k_rv_scatter  (seq, launch) records to their buckets, in any order
//   5. k_rv_rank     per bucket: a bitmap of its seq values in LDS; a launch's
//                    rank is the bucket's base plus the set bits below its own
// Seq values are unique, so the order inside a bucket needs no sort. The
// buckets are at most 2^18 values wide (all of 32 bits in 16384 buckets) and
// hold about a thousand launches each when seq is spread evenly; uneven seq
// only unbalances step 5. Equal seq values (an error, reported as ORDER) are
// seen there as a bit already set. A bucket of up to 4096 launches then counts
// the smaller (seq, launch) records for each; after a larger one the view is
// rebuilt by a stable radix sort in one block (k_rv_equal), which otherwise
// ends at once. Either way ties go by input index, as the general sort has it.
// 3M launches of 8 streams: 77 us (10 + 16 + 7 + 21 + 19 + 4), bound by the
// scatter's partial lines and by the latency of short kernels; the whole call
// 559 us with the sort, 375 us with this. 500k shuffled: 328 us and 229 us.
// Blocks of 256 and 1024 threads in step 5 and 2048 launches per bucket: the
// same within 3 us.
#include "common.h"
#include "impl.h"

namespace opa {

constexpr int kRvThreads = 1024, kRvPer = 8, kRvTile = kRvThreads * kRvPer;
constexpr int kRvPerBits = 10;  // log2 of the launches wanted per bucket
constexpr int kRvWords = (1 << kRvWidthBits) / 32;

struct RvArgs {
  const uint32_t *seq;
  int64_t T;
  uint32_t *mm;        // [0] smallest, [1] largest seq, [2] equal values seen
  uint32_t *cnt, *cur; // [kRvBuckets + 1] counts, then bases; next free place
  uint64_t *rec;       // [T] seq << 32 | launch, by bucket
  int32_t *sv, *rk;
  opattr_diag *diag;
  uint32_t *k0, *k1, *v0, *v1;  // [T] each: the sort of k_rv_equal (rec is k0 and k1)
};

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

__global__ void __launch_bounds__(kRvRankThreads) k_rv_rank(RvArgs a) {
  __shared__ uint32_t bits[kRvWords];
  __shared__ uint32_t tb[kRvRankThreads];  // set bits before each thread's words
  __shared__ uint32_t sh[kRvRankThreads / OPA_WAVE];
  __shared__ uint32_t equal;
  const int tid = threadIdx.x;
  const uint32_t lo = a.mm[0], hi = a.mm[1];
  const int shift = rv_shift(a, lo, hi);
  const uint32_t nb = ((hi - lo) >> shift) + 1u;
  const uint32_t words = shift > 5 ? 1u << (shift - 5) : 1u, mask = (1u << shift) - 1u;
  const uint32_t ch = (words + kRvRankThreads - 1) / kRvRankThreads;
  for (uint32_t b = blockIdx.x; b < nb; b += gridDim.x) {
    const uint32_t x0 = a.cnt[b], n = a.cnt[b + 1] - x0;
    if (n == 0) continue;  // uniform over the block
    const uint64_t *rec = a.rec + x0;
    for (uint32_t x = tid; x < words; x += kRvRankThreads) bits[x] = 0;
    if (tid == 0) equal = 0;
    __syncthreads();
    bool eq = false;
    for (uint32_t i0 = tid; i0 < n; i0 += kRvRankThreads * kRvUnroll) {
      uint32_t v[kRvUnroll];
#pragma unroll
      for (int k = 0; k < kRvUnroll; ++k) {
        const uint32_t i = i0 + k * kRvRankThreads;
        v[k] = i < n ? ((uint32_t)(rec[i] >> 32) - lo) & mask : 0u;
      }
#pragma unroll
      for (int k = 0; k < kRvUnroll; ++k)
        if (i0 + k * kRvRankThreads < n)
          eq |= (atomicOr(&bits[v[k] >> 5], 1u << (v[k] & 31)) >> (v[k] & 31)) & 1u;
    }
    if (eq) equal = 1;
    __syncthreads();
    if (equal) {  // uniform
      if (tid == 0) {
        if (n > kRvEqualMax) a.mm[2] = 1u;
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
      uint32_t c = 0;
      for (uint32_t k = 0; k < ch; ++k) {
        const uint32_t x = tid * ch + k;
        if (x < words) c += (uint32_t)__popc(bits[x]);
      }
      tb[tid] = x0 + block_excl_scan_add<uint32_t>(c, sh, nullptr);
      __syncthreads();
      for (uint32_t i0 = tid; i0 < n; i0 += kRvRankThreads * kRvUnroll) {
        uint64_t r[kRvUnroll];
#pragma unroll
        for (int k = 0; k < kRvUnroll; ++k) {
          const uint32_t i = i0 + k * kRvRankThreads;
          r[k] = i < n ? rec[i] : 0u;
        }
#pragma unroll
        for (int k = 0; k < kRvUnroll; ++k) {
          if (i0 + k * kRvRankThreads >= n) continue;
          const uint32_t v = ((uint32_t)(r[k] >> 32) - lo) & mask, wd = v >> 5;
          uint32_t q = tb[wd / ch] + (uint32_t)__popc(bits[wd] & ((1u << (v & 31)) - 1u));
          for (uint32_t x = wd / ch * ch; x < wd; ++x) q += (uint32_t)__popc(bits[x]);
          a.sv[q] = (int32_t)(uint32_t)r[k];
          a.rk[(uint32_t)r[k]] = (int32_t)q;
        }
      }
    }
    __syncthreads();  // the bitmap is free for the next bucket
  }
}

// Only after equal seq values: a stable sort of (seq, launch) in one block,
// 8 bits a pass, a tile of one pair per thread at a time.
__global__ void __launch_bounds__(kRvThreads) k_rv_equal(RvArgs a) {
  if (a.mm[2] == 0) return;  // uniform
  constexpr int kWaves = kRvThreads / OPA_WAVE;
  __shared__ uint32_t gb[256], wc[kWaves][256], sh[kWaves];
  const int tid = threadIdx.x, w = wave_id();
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 8 * pass;
    const uint32_t *ki = (pass & 1) ? a.k1 : a.k0, *vi = (pass & 1) ? a.v1 : a.v0;
    uint32_t *ko = (pass & 1) ? a.k0 : a.k1, *vo = (pass & 1) ? a.v0 : a.v1;
    auto key = [&](int64_t i) { return pass ? ki[i] : a.seq[i]; };
    if (tid < 256) gb[tid] = 0;
    __syncthreads();
    for (int64_t i = tid; i < a.T; i += kRvThreads) atomicAdd(&gb[(key(i) >> shift) & 255u], 1u);
    __syncthreads();
    const uint32_t g = tid < 256 ? gb[tid] : 0u;
    const uint32_t e = block_excl_scan_add<uint32_t>(g, sh, nullptr);
    if (tid < 256) gb[tid] = e;
    for (int64_t t0 = 0; t0 < a.T; t0 += kRvThreads) {
      for (int x = tid; x < kWaves * 256; x += kRvThreads) (&wc[0][0])[x] = 0;
      __syncthreads();
      const int64_t i = t0 + tid;
      const bool ok = i < a.T;
      const uint32_t k = ok ? key(i) : 0u, v = ok ? (pass ? vi[i] : (uint32_t)i) : 0u;
      const uint32_t d = (k >> shift) & 255u;
      const uint64_t pm = peers8(d) & __ballot(ok);
      const uint32_t lr = (uint32_t)__popcll(pm & lanemask_lt());
      if (ok && lr == 0) wc[w][d] = (uint32_t)__popcll(pm);
      __syncthreads();
      if (tid < 256) {
        uint32_t run = gb[tid];
        for (int x = 0; x < kWaves; ++x) {
          const uint32_t c = wc[x][tid];
          wc[x][tid] = run;
          run += c;
        }
        gb[tid] = run;
      }
      __syncthreads();
      if (ok) {
        const uint32_t dst = wc[w][d] + lr;
        ko[dst] = k;
        vo[dst] = v;
      }
      __syncthreads();
    }
    __threadfence_block();
    __syncthreads();
  }
  for (int64_t i = tid; i < a.T; i += kRvThreads) {  // four passes: back in k0, v0
    const uint32_t j = a.v0[i];
    a.sv[i] = (int32_t)j;
    a.rk[j] = (int32_t)i;
  }
}

size_t rank_view_entries() { return 2 * ((size_t)kRvBuckets + 64) + 64; }

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
  k_rv_equal<<<1, kRvThreads, 0, s>>>(a);
}

}  // namespace opa
