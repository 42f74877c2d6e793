// opattr_attribute for at most a million launches, in five launches on the
// caller's stream (before them, where it is not promised: the rank view of a
// seq with gaps, seven launches; the sort of the ranges, one and one for every
// merge pass; under OPATTR_VALIDATE the checks of the layout). Small calls are bound by the count of launches (5 us of
// host time each, two to three dozen of them) and by the chain of kernels,
// each of which takes 3 to 20 us however little it does; so every step does
// all the work that is ready, as jobs in disjoint block ranges of one grid:
//   1. k_c_pro   the launch-order view (sv[seq] = launch, dense seq), name
//                counts of every tile of profiled rows, validity and effective
//                ends of the ranges, their stream blocks, the clears
//   2. k_c_mid   per seq tile: key and in-tile rank of every launch, name
//                counts, partition edges; local parents of the ranges; prefix
//                of the profiled tiles' counts
//   3. k_c_join  parents in earlier tiles; slot table of the profiled rows;
//                prefix of the seq tiles' counts; partition records
//   4. k_c_tab / k_c_row   per block of launches as given: innermost range,
//                match with the dedup broadcast, and the reduction by operator
//                row (the table in LDS, or the launches ordered by row); depths
//                of the ranges; count validation
//   5. k_t_rows / k_c_rows  the table, the summary and the status
// Tiles hold one launch per thread of 1024-thread blocks (four past 256k
// launches, which then are one block per CU): the ranking of a tile of 4096 by
// 256 threads took 17 us by itself at any size.
#include "enclose_dev.h"
#include "match_dev.h"
#include "ranges_dev.h"
#include "rowagg.h"

namespace opa {

constexpr int kCThreads = kCompactTile;
constexpr int kCWaves = kCThreads / OPA_WAVE;
static_assert(kCThreads == kRlThreads, "the range tiles' threads");

struct CompactArgs {
  int64_t T, P;
  const uint32_t *seq, *name, *dur;
  const int32_t *part, *part_rep;  // NULL: no partitions
  const uint16_t *stream;
  const uint64_t *q;
  const int32_t *rk;  // launch-order rank of each launch; NULL: its seq
  int via;            // step 4 takes the launches by rank, not by position
  uint64_t *samp;     // every (1 << sshift)-th range start (via)
  int sshift;
  uint32_t NN, NP, NS, NOPS;
  int32_t *sv;   // launch at each rank
  uint32_t *kr;  // by rank: key << 16 | in-tile rank
  const uint32_t *pfname;
  int64_t nct, ncp;
  int tshift;  // log2 of the tiles' size
  uint32_t *tl, *pf;  // [tiles][NN] counts, then their prefixes
  uint32_t *tlc, *pfc, *off;
  int32_t *slot;
  uint32_t *pfirst, *plast, *pheads;
  PartRec *prec;
  RangeWork rw;
  int64_t *rblk;
  int32_t *match, *range_id;
  uint8_t *range_depth;
  uint32_t *name_counts;
  int skip_name, strict, validate, make_view;
  opattr_diag *diag;
  AggIn in;
  RowOut o;
  unsigned long long *tabs;  // [blocks][G][25] (table in LDS)
  unsigned long long *csum;  // [blocks][4] summary sums
  FillJobs fill;
  // blocks of each job, in grid order
  int j[6];
};

// job of block b: its number in jobs, and the block's index within it
__device__ __forceinline__ int job_of(const int (&j)[6], int b, int &i) {
  int n = 0;
#pragma unroll
  for (int k = 0; k < 5; ++k)
    if (n == k && b >= j[k]) {
      b -= j[k];
      n = k + 1;
    }
  i = b;
  return n;
}

// ---------------------------------------------------------------------------
// 1.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kCThreads) k_c_pro(CompactArgs a) {
  extern __shared__ __align__(16) unsigned char c_raw[];
  __shared__ uint32_t sbad;
  const int tid = threadIdx.x;
  int b;
  switch (job_of(a.j, (int)blockIdx.x, b)) {
    case 0: {  // a tile of profiled rows: its name counts
      uint32_t *cnt = reinterpret_cast<uint32_t *>(c_raw);
      if (tid == 0) sbad = 0;
      for (uint32_t n = tid; n < a.NN; n += kCThreads) cnt[n] = 0;
      __syncthreads();
      for (int64_t x = ((int64_t)b << a.tshift) + tid; x < (int64_t)(b + 1) << a.tshift; x += kCThreads)
        if (x < a.P) {
          const uint32_t n = a.pfname[x];
          if (n < a.NN) atomicAdd(&cnt[n], 1u);
          else atomicAdd(&sbad, 1u);
        }
      __syncthreads();
      for (uint32_t n = tid; n < a.NN; n += kCThreads) a.pf[(size_t)b * a.NN + n] = cnt[n];
      if (tid == 0 && sbad)
        atomicAdd((unsigned long long *)&a.diag->bad_records, (unsigned long long)sbad);
      break;
    }
    case 1: {  // validity and effective ends of the ranges
      const int64_t x = (int64_t)b * kCThreads + tid;
      count_bad(x < a.rw.cr.n && rprep_one(a.rw.cr, a.NS, a.NOPS, a.rw.ree, a.rw.npg, x), a.diag);
      if (a.via && x < a.rw.cr.n && (x & (((int64_t)1 << a.sshift) - 1)) == 0)
        a.samp[x >> a.sshift] = a.rw.cr.s[x];
      break;
    }
    case 2: {  // stream blocks of the ranges, one wave per stream s = 0..NS
      const uint32_t sw = (uint32_t)b * kCWaves + wave_id();
      if (sw <= a.NS) stream_block_wave(a.rw.cr.st, a.rw.cr.n, sw, a.rblk);
      break;
    }
    case 3: {  // the launch-order view (a false density promise leaves stale
               // entries in it: every reader checks their range; and launches
               // that no rank holds, which step 4 by rank leaves as here)
      const int64_t i = (int64_t)b * kCThreads + tid;
      bool bad = false;
      if (i < a.T) {
        if (a.via) a.match[i] = a.range_id[i] = -1;
        const uint32_t s = a.seq[i];
        if ((int64_t)s < a.T) a.sv[s] = (int32_t)i;
        else bad = a.validate != 0;
      }
      const uint64_t m = __ballot(bad);
      if (m && lane_id() == __ffsll((unsigned long long)m) - 1) {
        atomicAdd((unsigned long long *)&a.diag->order_violations, (unsigned long long)__popcll(m));
        atomicOr(&a.diag->flags, OPATTR_F_ORDER);
      }
      break;
    }
    case 4:  // the class map's range
      rep_check_one(a.part_rep, a.NP, a.diag, (uint32_t)b * kCThreads + tid);
      break;
    default: {  // the clears
      const int64_t stride = (int64_t)a.j[5] * kCThreads;
      for (int k = 0; k < a.fill.count; ++k)
        for (int64_t i = (int64_t)b * kCThreads + tid; i < a.fill.n[k]; i += stride)
          a.fill.p[k][i] = a.fill.v[k];
    }
  }
}

// ---------------------------------------------------------------------------
// 2. and 3.: ranks inside a tile, and prefixes down the tiles
// ---------------------------------------------------------------------------
// element c of the thread in a tile of CH elements per thread, in order along
// each wave's stretch
template <int CH>
__device__ __forceinline__ int c_elem(int c) {
  return wave_id() * (OPA_WAVE * CH) + c * OPA_WAVE + lane_id();
}

// In-tile ranks of the thread's elements with the given keys (keys >= NN are
// not ranked), the tile's counts in total (or NULL). cnt: kCWaves * NN entries
// of LDS. Called by the whole block.
template <int CH>
__device__ __forceinline__ void tile_rank(uint32_t (&key)[CH], uint32_t NN, uint16_t *cnt,
                                          uint32_t *total, uint32_t (&rank)[CH]) {
  const int w = wave_id();
  uint32_t *c32 = reinterpret_cast<uint32_t *>(cnt);
  for (uint32_t i = threadIdx.x; i < (kCWaves / 2) * NN; i += kCThreads) c32[i] = 0;
  __syncthreads();
  wave_rank<CH>(key, NN, bits_for(NN), cnt + (size_t)w * NN, rank);
  __syncthreads();
  for (uint32_t n = threadIdx.x; n < NN; n += kCThreads) {
    uint32_t run = 0;
#pragma unroll
    for (int v = 0; v < kCWaves; ++v) {
      const uint32_t c = cnt[(size_t)v * NN + n];
      cnt[(size_t)v * NN + n] = (uint16_t)run;
      run += c;
    }
    if (total) total[n] = run;
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < CH; ++c)
    if (key[c] < NN) rank[c] += cnt[(size_t)w * NN + key[c]];
}

// Exclusive prefix down 64 columns of a [rows][NN] table (rows <= 1024), in
// place, and the column totals: a wave per sixteenth of the rows.
__device__ __forceinline__ void tile_prefix(uint32_t *tab, int64_t rows, uint32_t NN, int cb,
                                            uint32_t *totals, uint32_t *sums) {
  constexpr int kB = 16;
  const int w = wave_id(), l = lane_id();
  const uint32_t col = (uint32_t)cb * OPA_WAVE + l;
  const int64_t per = (rows + kCWaves - 1) / kCWaves, r0 = w * per;
  const int64_t r1 = r0 + per < rows ? r0 + per : rows;
  uint32_t s = 0, v[kB];
  for (int64_t r = r0; r < r1; r += kB) {
#pragma unroll
    for (int i = 0; i < kB; ++i) v[i] = (col < NN && r + i < r1) ? tab[(r + i) * NN + col] : 0u;
#pragma unroll
    for (int i = 0; i < kB; ++i) s += v[i];
  }
  sums[w * OPA_WAVE + l] = s;
  __syncthreads();
  if (col >= NN) return;
  uint32_t run = 0;
  for (int k = 0; k < w; ++k) run += sums[k * OPA_WAVE + l];
  for (int64_t r = r0; r < r1; r += kB) {
    if (per > kB) {  // more than the batch that is still held
#pragma unroll
      for (int i = 0; i < kB; ++i) v[i] = r + i < r1 ? tab[(r + i) * NN + col] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kB; ++i)
      if (r + i < r1) {
        tab[(r + i) * NN + col] = run;
        run += v[i];
      }
  }
  if (w == kCWaves - 1) totals[col] = run;
}

// Key (name if eligible for replay, else NN) and partition (-1 none, -2 no
// launch or a bad id) of the launch at rank x; returns 1 for a bad id.
__device__ __forceinline__ uint32_t c_load(const CompactArgs &a, int64_t x, uint32_t &key,
                                           int32_t &lp) {
  key = a.NN;
  lp = -2;
  if (x < 0 || x >= a.T) return 0;
  const int32_t j = a.sv[x];
  if (j < 0 || (int64_t)j >= a.T) return 0;
  const uint32_t nm = a.name[j];
  const int32_t pt = a.part ? a.part[j] : -1;
  if (nm >= a.NN || pt < -1 || (pt >= 0 && (uint32_t)pt >= a.NP)) return 1;
  if (pt < 0 || a.part_rep[pt] == pt) key = nm;
  lp = pt;
  return 0;
}

template <int CH>  // launches per thread of a tile
__global__ void __launch_bounds__(kCThreads) k_c_mid(CompactArgs a) {
  extern __shared__ __align__(16) unsigned char c_raw[];
  const int tid = threadIdx.x;
  int b;
  switch (job_of(a.j, (int)blockIdx.x, b)) {
    case 0: {  // local parents of a tile of ranges
      int64_t *tree = reinterpret_cast<int64_t *>(c_raw);
      rlocal_tile(a.rw, b, tree, reinterpret_cast<int32_t *>(tree + kTreeNodes));
      break;
    }
    case 1: {  // a seq tile
      constexpr int kT = kCThreads * CH;
      __shared__ int32_t lp[kT + 2];  // partitions, with the neighbours'
      __shared__ uint32_t sbad;
      const int64_t base = (int64_t)b * kT;
      if (tid == 0) sbad = 0;
      uint32_t key[CH], r[CH], bad = 0;
      int32_t p[CH];
#pragma unroll
      for (int c = 0; c < CH; ++c) bad += c_load(a, base + c_elem<CH>(c), key[c], p[c]);
      if (a.pheads) {
#pragma unroll
        for (int c = 0; c < CH; ++c) lp[c_elem<CH>(c) + 1] = p[c];
        if (tid < 2) {
          uint32_t ek;
          int32_t e;
          c_load(a, tid == 0 ? base - 1 : base + kT, ek, e);
          lp[tid == 0 ? 0 : kT + 1] = e;
        }
      }
      tile_rank<CH>(key, a.NN, reinterpret_cast<uint16_t *>(c_raw), a.tl + (size_t)b * a.NN, r);
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int e = c_elem<CH>(c);
        const int64_t x = base + e;
        if (x < a.T) a.kr[x] = (key[c] << 16) | (key[c] < a.NN ? r[c] : 0u);
        if (a.pheads && p[c] >= 0) {  // partition edges: a head or a tail of a run
          if (lp[e] != p[c]) {
            a.pfirst[p[c]] = (uint32_t)x;
            atomicAdd(&a.pheads[p[c]], 1u);
          }
          if (lp[e + 2] != p[c]) a.plast[p[c]] = (uint32_t)x;
        }
      }
      const uint32_t bw = wave_reduce_add(bad);
      if (bw && lane_id() == 0) atomicAdd(&sbad, bw);
      __syncthreads();
      if (tid == 0 && sbad)
        atomicAdd((unsigned long long *)&a.diag->bad_records, (unsigned long long)sbad);
      break;
    }
    case 2:  // prefix of the profiled tiles' counts
      tile_prefix(a.pf, a.ncp, a.NN, b, a.pfc, reinterpret_cast<uint32_t *>(c_raw));
      break;
    default: {  // under OPATTR_VALIDATE: a launch that its own view entry does
                // not hold shares its seq with another
      const int64_t i = (int64_t)b * kCThreads + tid;
      bool bad = false;
      if (i < a.T) {
        const uint32_t s = a.seq[i];
        bad = (int64_t)s < a.T && a.sv[s] != (int32_t)i;
      }
      const uint64_t m = __ballot(bad);
      if (m && lane_id() == __ffsll((unsigned long long)m) - 1) {
        atomicAdd((unsigned long long *)&a.diag->order_violations, (unsigned long long)__popcll(m));
        atomicOr(&a.diag->flags, OPATTR_F_ORDER);
      }
    }
  }
}

template <int CH>
__global__ void __launch_bounds__(kCThreads) k_c_join(CompactArgs a) {
  extern __shared__ __align__(16) unsigned char c_raw[];
  __shared__ uint32_t sh[kCWaves];
  const int tid = threadIdx.x;
  int b;
  switch (job_of(a.j, (int)blockIdx.x, b)) {
    case 0:  // parents in earlier tiles
      rresolve_tree(a.rw, (int64_t)b * kCThreads, reinterpret_cast<int64_t *>(c_raw));
      break;
    case 1: {  // a tile of profiled rows into the slot table
      uint16_t *cnt = reinterpret_cast<uint16_t *>(c_raw);
      uint32_t *off = reinterpret_cast<uint32_t *>(cnt + (size_t)kCWaves * a.NN);
      static_assert(kCompactNames <= 2 * kCThreads, "two names a thread");
      const uint32_t n0 = 2u * tid;
      const uint32_t c0 = n0 < a.NN ? a.pfc[n0] : 0u, c1 = n0 + 1 < a.NN ? a.pfc[n0 + 1] : 0u;
      const uint32_t o0 = block_excl_scan_add<uint32_t>(c0 + c1, sh, nullptr);
      if (n0 < a.NN) off[n0] = o0;
      if (n0 + 1 < a.NN) off[n0 + 1] = o0 + c0;
      if (b == 0) {
        if (n0 < a.NN) a.off[n0] = o0;
        if (n0 + 1 < a.NN) a.off[n0 + 1] = o0 + c0;
      }
      const int64_t base = (int64_t)b * (kCThreads * CH);
      uint32_t key[CH], r[CH];
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int64_t x = base + c_elem<CH>(c);
        key[c] = x < a.P ? a.pfname[x] : a.NN;
        key[c] = key[c] < a.NN ? key[c] : a.NN;
      }
      tile_rank<CH>(key, a.NN, cnt, nullptr, r);
#pragma unroll
      for (int c = 0; c < CH; ++c)
        if (key[c] < a.NN)
          a.slot[off[key[c]] + a.pf[(size_t)b * a.NN + key[c]] + r[c]] =
              (int32_t)(base + c_elem<CH>(c));
      break;
    }
    case 2:  // prefix of the seq tiles' counts
      tile_prefix(a.tl, a.nct, a.NN, b, a.tlc, reinterpret_cast<uint32_t *>(c_raw));
      break;
    default:
      part_prep_one(a.part_rep, a.NP, a.pfirst, a.plast, a.pheads, a.prec, a.diag,
                    (uint32_t)b * kCThreads + tid);
  }
}

// ---------------------------------------------------------------------------
// 4. the launches as given
// ---------------------------------------------------------------------------
struct CFind {
  uint64_t red[2][kCWaves];
  int64_t win[2];
};
// the ranges that a block's main stream can need: start, end, parent, operator
struct CWin {
  uint64_t s[kCWindow];
  int64_t e[kCWindow];
  int32_t par[kCWindow];
  uint32_t op[kCWindow];
};

// The thread's kPer consecutive launches from ib on (nv of them exist; the
// block's first is i0): their outputs, match, duration and operator row
// (0xFFFFFFFF: no launch).
// The launches are taken by position where they come stream-major, else by
// launch-order rank through the view (kVia): launches near in launch order
// share operator rows, which keeps a block's partial results few, in whatever
// order they are given (500k shuffled launches over 1,001 rows by position:
// 480 rows in a block of 1024).
// Enclosure: the innermost range is the last one starting at or before the
// query point, or its first ancestor that ends at or after it. By position,
// the ranges between the smallest and largest query point of the block's main
// stream are staged in LDS, so that the search and the walk outward cost no
// memory round trips there; by rank, samples of all range starts are.
// Matching (see k_tl_look): the rank of the launch, or of the
// representative's launch at its position, among its name's eligible launches
// gives the profiled row. Its four levels of dependent loads are issued
// between the enclosure's, so that they cost no time of their own: a block's
// chain of memory round trips is what small calls wait for.
template <int kPer, int kThreads, bool kVia>
__device__ __forceinline__ void c_launches(const CompactArgs &a, int64_t i0, int64_t ib, int nv,
                                           CWin &win, CFind &sm, int32_t (&mt)[kPer],
                                           uint32_t (&du)[kPer], uint32_t (&g)[kPer]) {
  constexpr int kWaves = kThreads / OPA_WAVE;
  constexpr uint32_t kNone = 0xFFFFFFFFu;
  const int tid = threadIdx.x, w = wave_id(), ln = lane_id();
  uint32_t bad = 0, err = 0;
  // level 1: everything of the launches
  uint16_t st[kPer];
  uint64_t q[kPer];
  uint32_t sq[kPer], nm[kPer];
  int32_t pt[kPer], at_[kPer];
  bool ex[kPer];
  if constexpr (kVia) {
    load_n<kPer>(a.sv, ib, nv, at_);
    if (a.rw.cr.n > 0) {
      const int64_t ns = ((a.rw.cr.n - 1) >> a.sshift) + 1;
      for (int64_t k = tid; k < ns; k += kThreads) win.s[k] = a.samp[k];
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      // (a false density promise can leave any entry in the view)
      ex[k] = k < nv && at_[k] >= 0 && (int64_t)at_[k] < a.T;
      const int64_t i = ex[k] ? at_[k] : 0;
      st[k] = a.stream[i];
      q[k] = a.q[i];
      nm[k] = a.name[i];
      du[k] = ex[k] ? a.dur[i] : 0u;
      pt[k] = a.part ? a.part[i] : -1;
      sq[k] = (uint32_t)(ib + k);
    }
  } else {
    if constexpr (kPer == 1) {
      st[0] = nv > 0 ? a.stream[ib] : 0;
      q[0] = nv > 0 ? a.q[ib] : 0;
    } else {
      load_run<kPer>(a.stream, ib, nv, st);
      load_run<kPer>(a.q, ib, nv, q);
    }
    load_n<kPer>(a.rk ? reinterpret_cast<const uint32_t *>(a.rk) : a.seq, ib, nv, sq);
    load_n<kPer>(a.name, ib, nv, nm);
    if (a.part) load_n<kPer>(a.part, ib, nv, pt);
    load_n<kPer>(a.dur, ib, nv, du);
#pragma unroll
    for (int k = 0; k < kPer; ++k) ex[k] = k < nv;
  }
  const uint16_t s0 = kVia ? (uint16_t)0 : a.stream[i0];
  // level 2: partition records
  PartRec rc[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int32_t p = a.part ? pt[k] : -1;
    const bool ok = ex[k] && nm[k] < a.NN && (int64_t)sq[k] < a.T && p >= -1 &&
                    (p < 0 || (uint32_t)p < a.NP);
    rc[k] = PartRec{0, ok ? kRecEligible : kRecNone};
    if (ok && p >= 0) rc[k] = a.prec[p];
  }
  if constexpr (!kVia) {  // smallest and largest query point of the block's main stream
    uint64_t mn = ~0ull, mx = 0ull;
#pragma unroll
    for (int k = 0; k < kPer; ++k)
      if (ex[k] && st[k] == s0) {
        mn = q[k] < mn ? q[k] : mn;
        mx = q[k] > mx ? q[k] : mx;
      }
    for (int o = OPA_WAVE / 2; o > 0; o >>= 1) {
      const uint64_t y = __shfl_xor(mn, o, OPA_WAVE), z = __shfl_xor(mx, o, OPA_WAVE);
      mn = y < mn ? y : mn;
      mx = z > mx ? z : mx;
    }
    if (ln == 0) {
      sm.red[0][w] = mn;
      sm.red[1][w] = mx;
    }
  }
  // level 3: the rank that gives the row, and its name's place in the slots
  uint32_t kr[kPer], pre[kPer], rows[kPer], ro[kPer], dup = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    uint32_t src = kNone;
    const uint32_t hi = rc[k].hi;
    if (hi == kRecEligible) {
      src = sq[k];
    } else if (hi != kRecNone) {
      src = sq[k] + (uint32_t)rc[k].delta;
      dup |= 1u << k;
      if (sq[k] >= hi || (int64_t)src >= a.T) {
        src = kNone;
        err++;
      }
    }
    kr[k] = kNone;
    pre[k] = rows[k] = ro[k] = 0;
    if (src != kNone) {
      kr[k] = a.kr[src];
      pre[k] = a.tl[(size_t)(src >> a.tshift) * a.NN + nm[k]];
      rows[k] = a.pfc[nm[k]];
      ro[k] = a.off[nm[k]];
      if (a.skip_name && a.tlc[nm[k]] != rows[k]) rows[k] = 0;  // the name is left out
    }
  }
  __syncthreads();
  if constexpr (!kVia) {
    if (w < 2) {  // wave 0 finds the window's start, wave 1 its end
      uint64_t qa = ~0ull, qb = 0;
      for (int k = 0; k < kWaves; ++k) {
        qa = sm.red[0][k] < qa ? sm.red[0][k] : qa;
        qb = sm.red[1][k] > qb ? sm.red[1][k] : qb;
      }
      int64_t p = -1;
      if (s0 < a.NS && qa <= qb) {
        const int64_t lo = a.rblk[s0], hi = a.rblk[s0 + 1];
        p = wave_upper_bound(a.rw.cr.s, lo, hi, w == 0 ? qa : qb) - 1;
        if (w == 0 && p < lo) p = lo;
      }
      if (ln == 0) sm.win[w] = p;
    }
  }
  // level 4: the row
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    mt[k] = -1;
    if (kr[k] == kNone) continue;
    if ((kr[k] >> 16) != nm[k]) {  // the representative's launch has another name
      if ((dup >> k) & 1u) err++;
      continue;
    }
    const uint32_t r = pre[k] + (kr[k] & 0xFFFFu);
    if (r < rows[k]) mt[k] = a.slot[ro[k] + r];
  }
  int64_t wlo = 0, wn = 0;
  bool staged = false;
  if constexpr (!kVia) {
    __syncthreads();
    wlo = sm.win[0];
    wn = s0 < a.NS ? sm.win[1] - wlo + 1 : 0;
    if (wn < 0) wn = 0;
    staged = wn <= kCWindow;
    if (staged)
      for (int k = tid; k < wn; k += kThreads) {
        win.s[k] = a.rw.cr.s[wlo + k];
        win.e[k] = a.rw.ree[wlo + k];
        win.par[k] = a.rw.npg[wlo + k];
        win.op[k] = a.rw.cr.op[wlo + k];
      }
    __syncthreads();
  }
  const int32_t w0 = (int32_t)wlo, w1 = staged ? (int32_t)wn : 0;
  auto in_win = [&](int32_t j) { return !kVia && (uint32_t)(j - w0) < (uint32_t)w1; };
  int32_t pk[kPer], lok[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    pk[k] = -1;
    lok[k] = 0;
    if (ex[k] && st[k] < a.NS && q[k] < (1ull << 63)) {
      const int64_t lo = a.rblk[st[k]], hi = a.rblk[st[k] + 1];
      lok[k] = (int32_t)lo;
      if (!kVia && staged && st[k] == s0) {
        int l2 = 0, h2 = (int)wn;
        while (l2 < h2) {
          const int mid = (l2 + h2) >> 1;
          if (win.s[mid] <= q[k]) l2 = mid + 1;
          else h2 = mid;
        }
        const int64_t p = wlo + l2 - 1;
        pk[k] = (int32_t)(wn == 0 || p < lo ? lo - 1 : p);
      } else if constexpr (kVia) {
        // the samples inside the stream's block first, then between two of them
        const int sh = a.sshift;
        const int m0 = (int)((lo + ((int64_t)1 << sh) - 1) >> sh);
        int l2 = m0, h2 = hi > lo ? (int)((hi - 1) >> sh) + 1 : m0;
        while (l2 < h2) {
          const int mid = (l2 + h2) >> 1;
          if (win.s[mid] <= q[k]) l2 = mid + 1;
          else h2 = mid;
        }
        // every sample below l2 starts at or before the query point
        int64_t x0 = l2 > m0 ? (int64_t)(l2 - 1) << sh : lo, x1 = (int64_t)l2 << sh;
        x0 = x0 < lo ? lo : x0;
        x1 = x1 < hi ? x1 : hi;
        pk[k] = (int32_t)(thread_upper_bound(a.rw.cr.s, x0, x1, q[k]) - 1);
      } else {
        pk[k] = (int32_t)(thread_upper_bound(a.rw.cr.s, lo, hi, q[k]) - 1);
      }
    } else if (ex[k] && st[k] >= a.NS) {
      bad++;
    }
  }
  // up the parent chains, the thread's launches in lock step
  int64_t ek[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k)
    ek[k] = (ex[k] && pk[k] >= lok[k]) ? (in_win(pk[k]) ? win.e[pk[k] - w0] : a.rw.ree[pk[k]]) : 0;
  for (int step = 0; step < kMaxWalk; ++step) {
    bool act[kPer], any = false;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      act[k] = ex[k] && pk[k] >= lok[k] && ek[k] < (int64_t)q[k];
      any |= act[k];
    }
    if (!any) break;
#pragma unroll
    for (int k = 0; k < kPer; ++k)
      if (act[k]) pk[k] = in_win(pk[k]) ? win.par[pk[k] - w0] : a.rw.npg[pk[k]];
#pragma unroll
    for (int k = 0; k < kPer; ++k)
      if (act[k] && pk[k] >= lok[k])
        ek[k] = in_win(pk[k]) ? win.e[pk[k] - w0] : a.rw.ree[pk[k]];
  }
  int32_t rid[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    rid[k] = (ex[k] && pk[k] >= lok[k] && ek[k] >= (int64_t)q[k]) ? pk[k] : -1;
    g[k] = k < nv ? a.NOPS : 0xFFFFFFFFu;
    if (rid[k] >= 0) {
      g[k] = in_win(rid[k]) ? win.op[rid[k] - w0] : a.rw.cr.op[rid[k]];
      if (a.rw.cr.perm) rid[k] = a.rw.cr.perm[rid[k]];
    }
  }
  if constexpr (kVia) {
#pragma unroll
    for (int k = 0; k < kPer; ++k)
      if (ex[k]) {
        a.range_id[at_[k]] = rid[k];
        a.match[at_[k]] = mt[k];
      }
  } else {
    store_n<kPer>(a.range_id, ib, nv, rid);
    store_n<kPer>(a.match, ib, nv, mt);
  }
  const unsigned long long e = wave_reduce_add((unsigned long long)err);
  const uint32_t bb = wave_reduce_add(bad);
  if (ln == 0) {
    if (e) atomicAdd((unsigned long long *)&a.diag->dedup_errors, e);
    if (bb) atomicAdd((unsigned long long *)&a.diag->bad_records, (unsigned long long)bb);
  }
}

// the extra blocks of step 4: depths of the ranges, then the count validation
__device__ __forceinline__ void c_extra(const CompactArgs &a, int b) {
  if (b < a.j[1]) {
    const int64_t x = (int64_t)b * blockDim.x + threadIdx.x;
    range_depth_one(a.rw.npg, a.rw.ree, a.rw.cr.st, a.rw.cr.perm, a.rw.cr.n, a.NS, x,
                    a.range_depth, a.diag);
  } else {
    names_check(a.tlc, a.pfc, a.NN, a.name_counts, a.diag, a.strict);
  }
}

template <bool DEF, int kPer, bool kVia>
__global__ void __launch_bounds__(kTThreads) k_c_tab(CompactArgs a) {
  extern __shared__ __align__(16) unsigned char c_raw[];
  __shared__ CFind sm;
  __shared__ unsigned long long red[4][kCWaves];
  static_assert(kTThreads == kCThreads, "waves");
  if ((int)blockIdx.x >= a.j[0]) {
    c_extra(a, (int)blockIdx.x - a.j[0]);
    return;
  }
  const int tid = threadIdx.x;
  const int64_t i0 = (int64_t)blockIdx.x * (kTThreads * kPer), ib = i0 + (int64_t)tid * kPer;
  const int nv = (int)(a.T - ib < 0 ? 0 : (a.T - ib < kPer ? a.T - ib : kPer));
  int32_t mt[kPer];
  uint32_t du[kPer], g[kPer];
  c_launches<kPer, kTThreads, kVia>(a, i0, ib, nv, *reinterpret_cast<CWin *>(c_raw), sm, mt, du, g);
  unsigned long long *tab = reinterpret_cast<unsigned long long *>(c_raw);
  const uint32_t G = a.NOPS + 1u, ne = G * kFFields;
  __shared__ uint32_t turn[kTurns];
  __syncthreads();  // the window's space becomes the table
  for (uint32_t x = tid; x < ne; x += kTThreads) tab[x] = 0;
  if (tid < kTurns) turn[tid] = 0;
  __syncthreads();
  tab_add<DEF, kPer>(tab, turn, 0, a.in, nv, mt, du, g);
  __syncthreads();
  unsigned long long *dst = a.tabs + (size_t)blockIdx.x * ne;
  for (uint32_t x = tid; x < ne; x += kTThreads) dst[x] = tab[x];
  // the block's summary sums
  unsigned long long at_ = 0, un = 0, mt_ = 0;
  for (uint32_t r = tid; r < G; r += kTThreads) {
    const unsigned long long t = tab[(size_t)r * kFFields + 1];
    if (r < a.NOPS) at_ += t;
    else un += t;
    mt_ += tab[(size_t)r * kFFields + 3];
  }
  at_ = wave_reduce_add(at_);
  un = wave_reduce_add(un);
  mt_ = wave_reduce_add(mt_);
  if (lane_id() == 0) {
    red[0][wave_id()] = at_;
    red[1][wave_id()] = un;
    red[2][wave_id()] = at_ + un;
    red[3][wave_id()] = mt_;
  }
  __syncthreads();
  if (tid < 4) {
    unsigned long long v = 0;
    for (int k = 0; k < kCWaves; ++k) v += red[tid][k];
    a.csum[(size_t)blockIdx.x * 4 + tid] = v;
  }
}

template <bool DEF, int kPer, bool kVia>
__global__ void __launch_bounds__(kRThreads) k_c_row(CompactArgs a) {
  extern __shared__ __align__(16) unsigned char c_raw[];
  __shared__ CFind sm;
  __shared__ RowLds<kPer> lds;
  __shared__ unsigned long long red[3][kRThreads / OPA_WAVE];
  if ((int)blockIdx.x >= a.j[0]) {
    c_extra(a, (int)blockIdx.x - a.j[0]);
    return;
  }
  constexpr int kN = kRThreads * kPer;
  const int tid = threadIdx.x;
  const int64_t blk = blockIdx.x, i0 = blk * kN, ib = i0 + (int64_t)tid * kPer;
  const int nb = (int)(a.T - i0 < kN ? a.T - i0 : kN);
  const int nv = (int)(a.T - ib < 0 ? 0 : (a.T - ib < kPer ? a.T - ib : kPer));
  int32_t mt[kPer];
  uint32_t du[kPer], g[kPer];
  c_launches<kPer, kRThreads, kVia>(a, i0, ib, nv, *reinterpret_cast<CWin *>(c_raw), sm, mt, du, g);
  // the block's summary sums
  unsigned long long at_ = 0, un = 0, mt_ = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k)
    if (k < nv) {
      if (g[k] < a.NOPS) at_ += du[k];
      else un += du[k];
      if (mt[k] >= 0) mt_ += du[k];
    }
  at_ = wave_reduce_add(at_);
  un = wave_reduce_add(un);
  mt_ = wave_reduce_add(mt_);
  if (lane_id() == 0) {
    red[0][wave_id()] = at_;
    red[1][wave_id()] = un;
    red[2][wave_id()] = mt_;
  }
  __syncthreads();  // the window's space becomes the row histogram
  if (tid == 0) {
    unsigned long long v[3] = {0, 0, 0};
    for (int f = 0; f < 3; ++f)
      for (int k = 0; k < kRThreads / OPA_WAVE; ++k) v[f] += red[f][k];
    unsigned long long *c = a.csum + (size_t)blk * 4;
    c[0] = v[0];
    c[1] = v[1];
    c[2] = v[0] + v[1];
    c[3] = v[2];
  }
  const uint32_t words = r_hist_words(a.NOPS + 1u);
  uint32_t *hist = reinterpret_cast<uint32_t *>(c_raw);
  for (uint32_t x = tid; x < words; x += kRThreads) hist[x] = 0;
  row_order_block<DEF, kPer>(a.o, a.in, blk, nb, nv, mt, du, g, c_raw, lds);
}

// ---------------------------------------------------------------------------
// 5. the rows of a bucket from all blocks' partials and launch records; the
// unattributed row in a block of its own, then the finish. Every wave (or
// half wave, while the rows are few) adds to a copy of the rows of its own,
// and the copies are added up in pairs: a row in every block (the
// unattributed one above all) would otherwise take one addition after the
// other, 1500 of them for 180k launches, whose roundings add up (1.2e-15 of
// the table's 2-norm; 1.2e-16 with the copies, as a final rounding gives).
// ---------------------------------------------------------------------------
constexpr int kCRowThreads = 512, kCRowWaves = kCRowThreads / OPA_WAVE;
// copies of a bucket's rb rows (200 bytes each): 100 KB of LDS at most
__host__ __device__ inline int c_row_copies(uint32_t rb) {
  return rb <= 32 ? 2 * kCRowWaves : kCRowWaves;
}
static_assert(kFusedMaxRows / kBuckets <= 64, "the copies fit in LDS");

template <bool DEF>
__global__ void __launch_bounds__(kCRowThreads) k_c_rows(CombParams a) {
  constexpr int kPre = 2;
  extern __shared__ __align__(16) unsigned char c_raw[];
  __shared__ uint32_t list[kCRowWaves][kList];
  if (blockIdx.x > (unsigned)kBuckets) {
    finish_block(a.diag, a.sflag, a.ns, a.part, (int)a.nblocks, a.sum);
    return;
  }
  unsigned long long *tab = reinterpret_cast<unsigned long long *>(c_raw);  // [rows][kFFields]
  const uint32_t mx = DEF ? kDefMaxMask : a.mx, dw = DEF ? kDefDwMask : a.dw;
  const int tid = threadIdx.x, ln = lane_id(), w = wave_id();
  const uint32_t q = blockIdx.x;
  const bool un = q == (uint32_t)kBuckets;
  // rows [g0, g0 + nr): the bucket's, without the unattributed row
  const uint32_t g0 = un ? a.NOPS : q * a.rb;
  const uint32_t g1 = un ? a.G : (g0 + a.rb < a.NOPS ? g0 + a.rb : a.NOPS);
  if (g0 >= g1) return;
  const uint32_t nr = g1 - g0;
  const uint32_t ne = nr * kFFields;  // elements of a copy
  const int copies = c_row_copies(a.rb);
  for (uint32_t x = tid; x < ne * copies; x += kCRowThreads) tab[x] = 0;
  __syncthreads();
  unsigned long long *mine_tab =
      tab + (size_t)(copies == kCRowWaves ? w : 2 * w + (ln >> 5)) * ne;
  const int64_t per = (a.nblocks + kCRowWaves - 1) / kCRowWaves, b_lo = w * per;
  const int64_t b_hi = b_lo + per < a.nblocks ? b_lo + per : a.nblocks;
  for (int64_t b0 = b_lo; b0 < b_hi; b0 += (int64_t)OPA_WAVE * kPre) {
    comb_blocks<kPre>(mine_tab, un ? 1u : a.rb, list[w], a, q, b0, b_hi, mx, dw);
    wave_sync_lds();
  }
  __syncthreads();
  for (uint32_t x = tid; x < ne; x += kCRowThreads) {
    const int f = (int)(x % kFFields);
    unsigned long long v[2 * kCRowWaves];
#pragma unroll
    for (int k = 0; k < 2 * kCRowWaves; ++k) v[k] = k < copies ? tab[(size_t)k * ne + x] : 0ull;
    tab[x] = merge_tree(f, v, mx);  // only this thread reads element x of a copy
  }
  __syncthreads();
  for (uint32_t x = tid; x < nr * 24u; x += kCRowThreads) {
    const uint32_t r = x / 24u, o = x - r * 24u;
    reinterpret_cast<unsigned long long *>(a.table + g0 + r)[o] =
        row_field(tab + (size_t)r * kFFields, (int)o, a.absent, mx, dw);
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
#define OPA_C_LAUNCH(kernel, per, threads, lds)                                       \
  (a.via ? (def ? kernel<true, per, true><<<g, threads, lds, s>>>(a)                  \
                : kernel<false, per, true><<<g, threads, lds, s>>>(a))                \
         : (def ? kernel<true, per, false><<<g, threads, lds, s>>>(a)                 \
                : kernel<false, per, false><<<g, threads, lds, s>>>(a)))

static int blocks_of(int64_t n, int per) { return (int)((n + per - 1) / per); }

void run_compact(const CompactIn &x, hipStream_t s) {
  const Plan &pl = *x.pl;
  const opattr_kernels *k = x.k;
  const opattr_dims *d = x.d;
  void *ws = x.ws;
  const bool validate = (d->flags & OPATTR_VALIDATE) != 0;
  const bool parts = k->part_id && d->part_rep && d->n_parts > 0;
  check_kernel_layout(k, d, x.diag, s);
  if (!pl.seq_dense) build_seq_view(k, d, ws, pl, x.diag, validate, s);
  const CoreRanges cr = order_ranges(x.r, ws, pl, x.diag, validate, s);
  CompactArgs a{};
  a.T = pl.T;
  a.P = pl.P;
  a.seq = k->seq;
  a.name = k->name_id;
  a.dur = k->dur_ns;
  a.part = parts ? k->part_id : nullptr;
  a.part_rep = parts ? d->part_rep : nullptr;
  a.stream = k->stream_id;
  a.q = k->query_ns ? k->query_ns : k->start_ns;
  a.rk = pl.seq_dense ? nullptr : at<int32_t>(ws, pl.rk);
  a.via = (d->flags & OPATTR_KERNELS_STREAM_MAJOR) ? 0 : 1;
  a.samp = at<uint64_t>(ws, pl.csamp);
  while (pl.R > ((int64_t)kCWindow << a.sshift)) ++a.sshift;
  a.NN = pl.NN;
  a.NP = parts ? pl.NP : 0;
  a.NS = pl.NS;
  a.NOPS = d->n_ops;
  a.sv = at<int32_t>(ws, pl.sv);
  a.kr = at<uint32_t>(ws, pl.nbs);
  a.pfname = x.p->name_id;
  a.nct = pl.nct;
  a.ncp = pl.ncp;
  a.tshift = pl.ctshift;
  a.tl = at<uint32_t>(ws, pl.ctl);
  a.pf = at<uint32_t>(ws, pl.cpf);
  a.tlc = at<uint32_t>(ws, pl.tlc);
  a.pfc = at<uint32_t>(ws, pl.pfc);
  a.off = at<uint32_t>(ws, pl.off);
  a.slot = at<int32_t>(ws, pl.slot);
  a.pfirst = at<uint32_t>(ws, pl.pfirst);
  a.plast = at<uint32_t>(ws, pl.plast);
  a.pheads = parts ? at<uint32_t>(ws, pl.pheads) : nullptr;
  a.prec = at<PartRec>(ws, pl.prec);
  a.rw = range_work(cr, d, ws, pl, x.diag);
  a.rblk = at<int64_t>(ws, pl.rblk);
  a.match = x.match;
  a.range_id = x.range_id;
  a.range_depth = x.range_depth;
  a.name_counts = x.name_counts;
  a.skip_name = x.policy == OPATTR_MISMATCH_SKIP_NAME ? 1 : 0;
  a.strict = x.policy == OPATTR_MISMATCH_STRICT ? 1 : 0;
  a.validate = validate ? 1 : 0;
  a.make_view = pl.seq_dense ? 1 : 0;
  a.diag = x.diag;
  EncArgs e{};
  e.k = k;
  e.p = x.p;
  e.match = x.match;
  e.agg_kind = x.agg_kind;
  a.in = agg_inputs(e);
  a.o.NOPS = d->n_ops;
  a.o.rb = fused_rows_per_bucket(pl.G);
  a.o.parts = at<PartRow>(ws, pl.fparts);
  a.o.bkt = at<uint32_t>(ws, pl.fbkt);
  a.o.rec = at<uint4>(ws, pl.frec);
  a.o.pcap = (uint32_t)fused_part_cap(pl);
  a.o.rcap = (uint32_t)fused_span(pl);
  a.o.longrow = pl.flong;
  a.tabs = reinterpret_cast<unsigned long long *>(a.o.parts);
  a.csum = at<unsigned long long>(ws, pl.csum);
  a.fill.add(at<uint8_t>(ws, pl.sflag), 0, sflag_words(pl.NS));
  if (parts) {
    a.fill.add(a.pfirst, 0xFFFFFFFFu, pl.NP);
    a.fill.add(a.plast, 0xFFFFFFFFu, pl.NP);
    a.fill.add(a.pheads, 0u, pl.NP);
  }
  int64_t mx = 0;
  for (int q = 0; q < a.fill.count; ++q) mx = a.fill.n[q] > mx ? a.fill.n[q] : mx;
  const int ncol = blocks_of(pl.NN, OPA_WAVE), nbT = blocks_of(pl.T, kCThreads);
  const int nbR = blocks_of(pl.R, kCThreads), nbP = parts ? blocks_of(pl.NP, kCThreads) : 0;
  auto grid = [&](int j0, int j1, int j2, int j3, int j4, int j5) {
    const int v[6] = {j0, j1, j2, j3, j4, j5};
    int n = 0;
    for (int q = 0; q < 6; ++q) n += a.j[q] = v[q];
    return (unsigned)n;
  };
  const size_t lds_rank = (size_t)2 * kCWaves * pl.NN, lds_cols = (size_t)4 * kCThreads;
  const size_t lds_tree = (size_t)kTreeNodes * 8;
  auto most = [](size_t u, size_t v) { return u > v ? u : v; };
  probe_begin(OPATTR_PROBE_PF_HIST, s);
  unsigned g = grid((int)pl.ncp, nbR, blocks_of((int64_t)pl.NS + 1, kCWaves), a.make_view ? nbT : 0,
                    nbP, blocks_of(mx, kCThreads) < 256 ? blocks_of(mx, kCThreads) : 256);
  k_c_pro<<<g, kCThreads, (size_t)4 * pl.NN, s>>>(a);
  probe_end(OPATTR_PROBE_PF_HIST, s);
  probe_begin(OPATTR_PROBE_TL_HIST, s);
  g = grid(pl.R > 0 ? (int)pl.ntr_max : 0, (int)pl.nct, ncol,
           validate && a.make_view ? nbT : 0, 0, 0);
  const size_t lds_mid = most(most(lds_rank, lds_cols), lds_tree + (kInlineBases + 1) * 4);
  const bool one = pl.ctshift == 10;  // one launch per thread of a tile, else four
  if (one) k_c_mid<1><<<g, kCThreads, lds_mid, s>>>(a);
  else k_c_mid<4><<<g, kCThreads, lds_mid, s>>>(a);
  probe_end(OPATTR_PROBE_TL_HIST, s);
  probe_begin(OPATTR_PROBE_RANGES, s);
  g = grid(nbR, (int)pl.ncp, ncol, nbP, 0, 0);
  const size_t lds_join = most(most(lds_rank + (size_t)4 * pl.NN, lds_cols), lds_tree);
  if (one) k_c_join<1><<<g, kCThreads, lds_join, s>>>(a);
  else k_c_join<4><<<g, kCThreads, lds_join, s>>>(a);
  probe_end(OPATTR_PROBE_RANGES, s);
  const bool def = a.in.maxmask == kDefMaxMask && a.in.dwmask == kDefDwMask;
  CombParams c{};
  c.rb = a.o.rb;
  c.G = pl.G;
  c.NOPS = d->n_ops;
  c.mx = a.in.maxmask;
  c.dw = a.in.dwmask;
  c.absent = x.p->absent_mask;
  c.parts = a.o.parts;
  c.bkt = a.o.bkt;
  c.pcap = a.o.pcap;
  c.rec = a.o.rec;
  c.rcap = a.o.rcap;
  c.in = a.in;
  c.table = x.table;
  c.part = a.csum;
  c.diag = x.diag;
  c.sflag = at<uint8_t>(ws, pl.sflag);
  c.ns = d->n_streams;
  c.sum = x.sum;
  c.nblocks = fused_agg_blocks(pl.T, fused_span(pl));
  probe_begin(OPATTR_PROBE_MAIN_PASS, s);
  if (pl.ftabs) {
    const size_t lt = most(fused_tab_bytes(pl.G), sizeof(CWin));
    g = grid(pl.ftabs, nbR, 1, 0, 0, 0);
    if (pl.fper == 1) OPA_C_LAUNCH(k_c_tab, 1, kTThreads, lt);
    else if (pl.fper == 2) OPA_C_LAUNCH(k_c_tab, 2, kTThreads, lt);
    else OPA_C_LAUNCH(k_c_tab, 4, kTThreads, lt);
  } else {
    const size_t lr = most(r_agg_lds(pl.G, pl.fper, pl.flong), sizeof(CWin));
    g = grid((int)c.nblocks, blocks_of(pl.R, kRThreads), 1, 0, 0, 0);
    if (pl.fper == 2) OPA_C_LAUNCH(k_c_row, 2, kRThreads, lr);
    else OPA_C_LAUNCH(k_c_row, 4, kRThreads, lr);
  }
  probe_end(OPATTR_PROBE_MAIN_PASS, s);
  probe_begin(OPATTR_PROBE_AGGREGATE, s);
  if (pl.ftabs) {
    const unsigned gr = (pl.G + kTRows - 1) / kTRows + 1;
    if (def) k_t_rows<true, false><<<gr, 1024, 0, s>>>(c, a.tabs, pl.ftabs);
    else k_t_rows<false, false><<<gr, 1024, 0, s>>>(c, a.tabs, pl.ftabs);
  } else {
    const size_t lt = (size_t)c_row_copies(a.o.rb) * a.o.rb * kFFields * 8;
    if (def) k_c_rows<true><<<kBuckets + 2, kCRowThreads, lt, s>>>(c);
    else k_c_rows<false><<<kBuckets + 2, kCRowThreads, lt, s>>>(c);
  }
  probe_end(OPATTR_PROBE_AGGREGATE, s);
}

}  // namespace opa
