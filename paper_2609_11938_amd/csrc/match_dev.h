// Device code of the matching shared by its own kernels and the compact path's
// multi-job kernels.
#pragma once
#include "common.h"
#include "impl.h"

namespace opa {

// count validation (Sec. 3.3): per name, eligible launches against rows;
// run by one block of up to 1024 threads
__device__ inline void names_check(const uint32_t *__restrict__ tlc, const uint32_t *__restrict__ pfc,
                            uint32_t NN, uint32_t *name_counts, opattr_diag *diag, int strict) {
  __shared__ unsigned long long red[3][16];
  unsigned long long mism = 0, tlu = 0, pfu = 0;
  for (uint32_t n = threadIdx.x; n < NN; n += blockDim.x) {
    const uint32_t tl = tlc[n], pf = pfc[n];
    if (name_counts) {
      name_counts[2 * (size_t)n] = tl;
      name_counts[2 * (size_t)n + 1] = pf;
    }
    if (tl != pf) {
      mism++;
      if (tl > pf) tlu += tl - pf;
      else pfu += pf - tl;
    }
  }
  mism = wave_reduce_add(mism);
  tlu = wave_reduce_add(tlu);
  pfu = wave_reduce_add(pfu);
  if (lane_id() == 0) {
    red[0][wave_id()] = mism;
    red[1][wave_id()] = tlu;
    red[2][wave_id()] = pfu;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long a = 0, b = 0, c = 0;
    for (uint32_t i = 0; i < blockDim.x / OPA_WAVE; ++i) {
      a += red[0][i];
      b += red[1][i];
      c += red[2][i];
    }
    if (a) {
      atomicAdd(&diag->names_mismatched, (uint32_t)a);
      atomicOr(&diag->flags, OPATTR_F_COUNT);
    }
    if (b) atomicAdd((unsigned long long *)&diag->tl_unmatched, b);
    if (c) atomicAdd((unsigned long long *)&diag->pf_unmatched, c);
    if (strict) diag->strict = 1u;
  }
}

// The record of partition p (PartRec, see impl.h); also raises PARTITION when
// it is seen in more than one run. Called by whole waves.
__device__ inline void part_prep_one(const int32_t *part_rep, uint32_t NP, const uint32_t *pfirst,
                                     const uint32_t *plast, const uint32_t *pheads, PartRec *prec,
                                     opattr_diag *diag, uint32_t p) {
  bool nc = false;
  if (p < NP) {
    nc = pheads[p] > 1;
    if (prec) {
      const int32_t r = part_rep[p];
      PartRec q{0, kRecNone};
      if (r == (int32_t)p) {
        q.hi = kRecEligible;
      } else if (r >= 0 && (uint32_t)r < NP) {
        q.hi = 0;
        const uint32_t f = pfirst[r];
        if (pheads[p] == 1u && pheads[r] == 1u && part_rep[r] == r && f != 0xFFFFFFFFu) {
          q.delta = (int32_t)(f - pfirst[p]);
          const uint64_t hi = (uint64_t)pfirst[p] + (plast[r] - f + 1u);
          q.hi = (uint32_t)(hi < 0x7FFFFFFFull ? hi : 0x7FFFFFFFull);  // seq ranks are < 2^31
        }
      }
      prec[p] = q;
    }
  }
  if (__ballot(nc) && lane_id() == 0) atomicOr(&diag->flags, OPATTR_F_PARTITION);
}

// class map entry q in range, else a bad record; called by whole waves
__device__ __forceinline__ void rep_check_one(const int32_t *part_rep, uint32_t NP,
                                              opattr_diag *diag, uint32_t q) {
  const bool bad = q < NP && (part_rep[q] < 0 || (uint32_t)part_rep[q] >= NP);
  const uint64_t m = __ballot(bad);
  if (m && lane_id() == __ffsll((unsigned long long)m) - 1)
    atomicAdd((unsigned long long *)&diag->bad_records, (unsigned long long)__popcll(m));
}

// The processing order of the run reduction's nb blocks of span launches, by
// the seq rank of each block's first launch (a counting sort into windows).
// One block of kOrderBuckets threads; hist holds kOrderBuckets entries, sh
// one per wave.
constexpr int kOrderBuckets = 1024;
__device__ inline void block_order(const uint32_t *__restrict__ seq, int64_t T, int64_t nb,
                                   int span, uint32_t *order, uint32_t *hist, uint32_t *sh) {
  const int tid = threadIdx.x;
  hist[tid] = 0;
  __syncthreads();
  auto bucket = [&](int64_t b) -> uint32_t {
    const uint64_t q = seq[b * span];
    const uint64_t c = q < (uint64_t)T ? q : (uint64_t)T - 1;  // a broken promise: any window
    return (uint32_t)(c * kOrderBuckets / (uint64_t)T);
  };
  for (int64_t b = tid; b < nb; b += kOrderBuckets) atomicAdd(&hist[bucket(b)], 1u);
  __syncthreads();
  uint32_t tot;
  const uint32_t base = block_excl_scan_add<uint32_t>(hist[tid], sh, &tot);
  __syncthreads();
  hist[tid] = base;
  __syncthreads();
  for (int64_t b = tid; b < nb; b += kOrderBuckets)
    order[atomicAdd(&hist[bucket(b)], 1u)] = (uint32_t)b;
}

}  // namespace opa
