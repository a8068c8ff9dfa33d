// The per-request plan by one wave, a request per lane, for batches of at most kLanePlanReqs
// requests: the plan kernel's work for such batches, and what the first kernel of a call does for
// itself so that no plan kernel precedes it (a launch of its own costs 4-6 us on MI355X, mostly
// ramp and dependent loads, before the kernel that reads the plan can start; the scans here cost
// about half a microsecond, beside loads that the reading kernel waited for in any case).
#pragma once

#include "device_common.hpp"

namespace actkv {

// Exclusive prefix sum over the wave.
__device__ __forceinline__ int64_t wave_excl_scan_i64(int64_t v) { return wave_incl_scan_i64(v) - v; }

// Request `lane` of the batch (zeros past R) and the sums over the requests before it.
struct LanePlan {
  int32_t L, n;
  int32_t q_off;      // sum of n
  int64_t seg_off;    // Hkv * sum of L
  int64_t tiles;      // key tiles
  int64_t cost;       // scoring cost
  int64_t own_cost;   // of this request
};

// Row chunks of a request and the scoring cost of one key tile of chunk c.
__device__ __forceinline__ int lane_chunks(int G, int n) {
  return n > 0 ? ceil_div(G * n, kRowsPerChunk) : 1;
}
__device__ __forceinline__ int64_t lane_tile_cost(int G, int n, int c) {
  return score_tile_cost(chunk_units((int64_t)G * n - (int64_t)c * kRowsPerChunk));
}

__device__ __forceinline__ LanePlan lane_plan(const DevProblem& dp) {
  const int r = threadIdx.x & 63;
  LanePlan p;
  p.L = r < dp.R ? dp.seq_lens[r] : 0;
  p.n = r < dp.R ? dp.q_lens[r] : 0;
  const int64_t ntiles = ceil_div64(p.L, kKeyTile);
  int64_t per_tile = lane_tile_cost(dp.G, p.n, 0);
  if (dp.max_chunks > 1) {   // every chunk but the last costs what the first does
    const int chunks = lane_chunks(dp.G, p.n);
    if (chunks > 1) per_tile = per_tile * (chunks - 1) + lane_tile_cost(dp.G, p.n, chunks - 1);
  }
  p.own_cost = r < dp.R ? ntiles * per_tile * dp.Hkv : 0;
  p.q_off = (int32_t)wave_excl_scan_i64(p.n);
  p.seg_off = wave_excl_scan_i64((int64_t)p.L * dp.Hkv);
  p.tiles = wave_excl_scan_i64(ntiles);
  p.cost = wave_excl_scan_i64(p.own_cost);
  return p;
}

// What request `lane`'s budgets decide: entries kept over its heads and whether it is left alone,
// fresh and freed pages (see plan_kernel), and the sums over the requests before it.
struct LaneBudgets {
  int64_t kept, kept_off;
  int32_t skip, X, Y;
  int32_t fresh_off, freed_off;
};

__device__ __forceinline__ LaneBudgets lane_budgets(const DevProblem& dp, const LanePlan& lp) {
  const int r = threadIdx.x & 63, Hkv = dp.Hkv;
  const bool ok = r < dp.R;
  const int32_t L = lp.L;
  int32_t kmax = 0, bmin = INT32_MAX;
  LaneBudgets b;
  b.kept = 0;
  // budgets 8 at a time, every load of a batch issued before any is used
  for (int h0 = 0; h0 < Hkv; h0 += 8) {
    int32_t bb[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) bb[u] = ok && h0 + u < Hkv ? dp.budgets[r * Hkv + h0 + u] : INT32_MAX;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (h0 + u >= Hkv) break;
      const int32_t k = bb[u] < L ? bb[u] : L;
      b.kept += k;
      kmax = k > kmax ? k : kmax;
      bmin = bb[u] < bmin ? bb[u] : bmin;
    }
  }
  b.skip = bmin >= L;
  b.X = b.skip ? 0 : ceil_div(kmax, kPageSize);
  b.Y = b.skip ? 0 : ceil_div(L, kPageSize);
  b.kept_off = wave_excl_scan_i64(b.kept);
  b.fresh_off = (int32_t)wave_excl_scan_i64(b.X);
  b.freed_off = (int32_t)wave_excl_scan_i64(b.Y);
  return b;
}

// Request r's plan from the lanes; the scoring and LSE fields are left 0.
__device__ __forceinline__ ReqPlan lane_request(const LanePlan& lp, const LaneBudgets& lb, int r) {
  ReqPlan p = {};
  p.L = __builtin_amdgcn_readlane(lp.L, r);
  p.n = __builtin_amdgcn_readlane(lp.n, r);
  p.X = __builtin_amdgcn_readlane(lb.X, r);
  p.Y = __builtin_amdgcn_readlane(lb.Y, r);
  p.skip = __builtin_amdgcn_readlane(lb.skip, r);
  p.q_off = __builtin_amdgcn_readlane(lp.q_off, r);
  p.fresh_off = __builtin_amdgcn_readlane(lb.fresh_off, r);
  p.freed_off = __builtin_amdgcn_readlane(lb.freed_off, r);
  p.seg_off = readlane_i64(lp.seg_off, r);
  return p;
}

// Where the kept entries of (r, h) start (a head per lane: at most 64 of them).
__device__ __forceinline__ int64_t lane_kept_off(const DevProblem& dp, const ReqPlan& pl,
                                                 const LaneBudgets& lb, int r, int h) {
  const int u = threadIdx.x & 63;
  const int32_t b = u < h ? dp.budgets[r * dp.Hkv + u] : 0;
  return readlane_i64(lb.kept_off, r) +
         readlane_i64(wave_incl_scan_i64(b < pl.L ? b : pl.L), kWave - 1);
}

// The workspace's plan of the whole batch, from the lanes of one wave.
__device__ __forceinline__ void write_plan(const DevProblem& dp, const LanePlan& lp) {
  const int r = threadIdx.x & 63, Hkv = dp.Hkv, C = dp.max_chunks;
  const bool ok = r < dp.R;
  const int32_t L = lp.L;
  const LaneBudgets lb = lane_budgets(dp, lp);
  const int32_t lse_blocks = (int32_t)ceil_div64(L, kLseKeysPerBlock);
  const int64_t l_off = wave_excl_scan_i64((int64_t)lp.n * dp.Hq * lse_blocks);
  const int64_t f_off = wave_excl_scan_i64(lb.Y - lb.X);
  const int nchunk = lane_chunks(dp.G, lp.n);
  if (ok) {
    ReqPlan p;
    p.L = L; p.n = lp.n; p.X = lb.X; p.Y = lb.Y; p.skip = lb.skip; p.nchunk = nchunk;
    p.q_off = lp.q_off; p.fresh_off = lb.fresh_off; p.freed_off = lb.freed_off;
    p.lse_blocks = lse_blocks; p.seg_off = lp.seg_off; p.lse_part_off = l_off;
    p.ip_freed_off = (int32_t)f_off;
    dp.plan[r] = p;
    dp.req_done[r] = 0;
    // kept offsets per (r, h)
    int64_t ko = lb.kept_off;
    for (int h0 = 0; h0 < Hkv; h0 += 8) {
      int32_t bb[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) bb[u] = h0 + u < Hkv ? dp.budgets[r * Hkv + h0 + u] : 0;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (h0 + u >= Hkv) break;
        dp.kept_off[r * Hkv + h0 + u] = ko;
        ko += bb[u] < L ? bb[u] : L;
      }
    }
    // scoring cost prefix per segment (r, c, h), c < max_chunks
    const int64_t ntiles = ceil_div64(L, kKeyTile);
    int64_t co = lp.cost;
    for (int c = 0; c < C; ++c) {
      const int64_t step = c < nchunk ? ntiles * lane_tile_cost(dp.G, lp.n, c) : 0;
      for (int h = 0; h < Hkv; ++h) {
        dp.seg_cost[((int64_t)r * C + c) * Hkv + h] = co;
        co += step;
      }
    }
  }
  if (r == 63) {
    dp.kept_off[(int64_t)dp.R * Hkv] = lb.kept_off + lb.kept;
    dp.seg_cost[dp.num_segments] = lp.cost + lp.own_cost;
    *dp.plan_sig = dp.sig;   // the plan now belongs to this problem
  }
}

}  // namespace actkv
