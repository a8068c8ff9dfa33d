// The block-table rewrite of the fresh-page compaction, by one workgroup.
#pragma once

#include "device_common.hpp"

namespace actkv {

constexpr int kRewriteBatch = 8;   // block-table entries a rewrite thread reads together

// Request r's block-table rewrite: new lengths, the old row to the freed list, the fresh
// pages (then -1) into the row.  Runs after every read of the old row.
__device__ __forceinline__ void rewrite_row(const DevProblem& dp, int r, const ReqPlan& pl,
                                            int32_t* bt, const int32_t* __restrict__ free_pages,
                                            int32_t* __restrict__ freed,
                                            int32_t* __restrict__ new_lens) {
  const int Hkv = dp.Hkv;
  for (int h = threadIdx.x; h < Hkv; h += blockDim.x) {
    const int b = dp.budgets[r * Hkv + h];
    new_lens[r * Hkv + h] = pl.skip ? pl.L : (b < pl.L ? b : pl.L);
  }
  if (pl.skip || pl.Y <= 0) return;
  // batches of kRewriteBatch entries per thread: every load of a batch is issued before its
  // stores (an entry is read and written by the same thread only), and the loads carry no
  // condition (indices past the row re-read its last entry, values unused), so they are in
  // flight together instead of one round trip per entry
  int32_t* row = bt + (int64_t)r * dp.bt_stride;
  const int last = pl.Y - 1;
  // the fresh page ids (a request that takes none, every head keeping nothing, reads its own
  // row instead and writes -1)
  const int32_t* fresh = pl.X > 0 ? free_pages + pl.fresh_off : row;
  const int fresh_last = pl.X > 0 ? pl.X - 1 : last;
  for (int i0 = threadIdx.x; i0 < pl.Y; i0 += kRewriteBatch * (int)blockDim.x) {
    int32_t old[kRewriteBatch], now[kRewriteBatch];
#pragma unroll
    for (int u = 0; u < kRewriteBatch; ++u) {
      const int i = i0 + u * (int)blockDim.x;
      old[u] = row[i < last ? i : last];
      now[u] = fresh[i < fresh_last ? i : fresh_last];
    }
#pragma unroll
    for (int u = 0; u < kRewriteBatch; ++u) {
      const int i = i0 + u * (int)blockDim.x;
      if (i < pl.Y) {
        freed[pl.freed_off + i] = old[u];
        row[i] = i < pl.X ? now[u] : -1;
      }
    }
  }
}

}  // namespace actkv
