// A segment's selection by one 1024-thread workgroup with the keys in registers (segments up to
// kRegMaxLen entries, pooling windows up to 2 * kPoolHalo + 1).  Included by select.hip inside
// its namespaces, after the shared building blocks.
//
// Layout: the segment is cut into groups of 64 entries; wave w holds groups w * per ..
// w * per + per - 1, one entry per lane and one register per group (`per` <= NG registers, the
// template argument).  Loads and stores of a group are coalesced, a comparison of a group is one
// instruction that leaves its 64 answers in a scalar mask, and positions in the output come from
// counting mask bits.
//
// One workgroup's four SIMDs are what bounds the selection (128 segments of a 32-request batch
// leave half the CUs without one): an instruction per entry costs 0.23 us at 35,000 entries.
// So every entry is looked at as few times as an exact answer allows:
//   pool     the raw keys pass through LDS 8 groups at a time (private to the wave, no barrier)
//            and meet their window's neighbours there
//   bracket  at most kSamples of the pooled keys (spread over the segment) bound the k-th largest
//            key from both sides: a histogram of the sample across the segment's key range
//   count    entries above the bracket are counted, those inside go to a histogram of 1,024 bins
//            across it: one in six or so makes an LDS atomic, into as many bins
//   choose   the bin with the k-th entry: its few entries are listed and ranked against each other,
//            which gives the last entry taken (its key and its index)
//   emit     one mask per group gives the kept indices in ascending order
// When the bracket turns out not to hold the k-th entry the count is repeated over the whole key
// range, and when the chosen bin holds more than the list does, over that bin: the result is exact
// for every input, and ordinary scores need one pass.
//
// Replaces radix passes over runs of consecutive entries per thread (keys in LDS, or in registers
// past 38,400 entries): see the figures at select_kernel.

constexpr int kRegWaves = kSelectThreads / 64;
constexpr int kRegChunk = 8;                     // groups that meet in LDS at a time
constexpr int kRegChunkWords = kRegChunk * 64 + 2 * kPoolHalo;
constexpr int kRegMaxGroups = 63;                // per wave
constexpr int kRegMaxLen = kRegMaxGroups * kSelectThreads;   // 64,512
static_assert(kRegMaxLen == kLrfuMaxLen && 2 * kPoolHalo + 1 == kLrfuRegMaxWindow,
              "the LRFU selection's limits are those of the register-resident path");
constexpr int kSamples = kSelectThreads;         // sample slots: one per thread
constexpr int kCells = kSelectThreads;           // histogram bins: one per thread
// Entries of the chosen bin that are ranked, one per lane of a wave; a fuller bin is cut into bins
// again.  Ordinary scores leave a few.  (Up to 1,024, an entry per thread against all the others: the
// 900 equal entries of a bin, 35,000 scores of 40 values, took LRFU to 230 us against 92 with 64 and
// 108 with radix passes.)
constexpr int kListMax = 64;

struct RegLds {
  union {
    uint32_t chunk[kRegWaves][kRegChunkWords];   // pooling
    struct {
      union {
        uint32_t hist[kCells];
        uint64_t mass[kCells];                   // the LRFU top-p search
      };
      uint32_t samp[kSamples];
      uint32_t list_key[kListMax];
      int32_t list_at[kListMax];
    };
  };
  int64_t scan[17];
  uint64_t sum[2 * kRegWaves];
  float cut_value;
  uint32_t range[2 * kRegWaves];                 // the waves' largest keys, and complements of the smallest
  uint32_t bracket[2];
  int bin, listed;
  uint32_t bin_count;
  uint64_t bin_need;
  uint32_t last_key;                             // the last entry taken
  int32_t last_at;
};

struct RegGeom {
  int L, per, w, lane;   // entries, groups per wave, this wave and lane
  int start, n;          // the wave's first entry and how many it has
  __device__ __forceinline__ int first() const { return start + lane; }   // entry of slot 0
};

__device__ __forceinline__ RegGeom reg_geom(int L) {
  RegGeom g;
  g.L = L;
  g.per = (L + kSelectThreads - 1) / kSelectThreads;
  g.w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  g.lane = (int)threadIdx.x & 63;
  g.start = g.w * g.per * 64;
  const int left = L - g.start;
  g.n = left < 0 ? 0 : (left < g.per * 64 ? left : g.per * 64);
  return g;
}

// The slots that hold an entry: lane i gets the mask of the wave's slot i.  The others hold key 0,
// which one NaN's key is too (0xFFFFFFFF), and past `per` their indices are the next wave's: what is
// counted or taken among keys of 0 goes through this mask.
__device__ __forceinline__ uint64_t reg_real(const RegGeom& g) {
  const int n = g.n - g.lane * 64;
  return n <= 0 ? 0ull : (n >= 64 ? ~0ull : (1ull << n) - 1ull);
}

// f(b, i) for slots i = 8 b .. 8 b + 7 (below NG) of every chunk b in use.  Only chunks are skipped
// (a scalar branch per chunk; one per slot cost a scalar register pair each, kept across the
// kernel): slots past the wave's entries hold key 0.
template <int NG, typename F>
__device__ __forceinline__ void for_slots(const RegGeom& g, F f) {
#pragma unroll
  for (int b = 0; b < (NG + kRegChunk - 1) / kRegChunk; ++b) {
    if (b * kRegChunk >= g.per) continue;
#pragma unroll
    for (int j = 0; j < kRegChunk; ++j)
      if (b * kRegChunk + j < NG) f(b, b * kRegChunk + j);
  }
}

// Orders the wave's LDS writes before its later LDS reads of what other lanes wrote (the wave's
// LDS accesses are carried out in order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Wave-wide maximum (every lane gets it).
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// order_key of a raw score's bits (x + 0 makes a zero of either sign +0).
__device__ __forceinline__ uint32_t bits_key(uint32_t bits) {
  const uint32_t u = __float_as_uint(__uint_as_float(bits) + 0.0f);
  return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

// Added to order keys, this puts every NaN's (past +inf's, and below -inf's) below all the others,
// +inf's being the largest: while the scores are pooled a NaN then yields to its neighbours, as it does
// to fmaxf on the other paths.
constexpr uint32_t kPoolBias = 0x007FFFFFu;

// The order keys of the segment's max-pooled scores: r[i] for the entry of slot i, 0 (below every
// score's key) past the wave's entries.  Pooled scores to pout when given.
template <int NG>
__device__ __forceinline__ void reg_load_pooled(const RegGeom g, int hw,
                                                const float* __restrict__ in, float* pout,
                                                RegLds& lds, uint32_t (&r)[NG]) {
  constexpr int kChunks = (NG + kRegChunk - 1) / kRegChunk;
  // the wave's own entries: slots past them read 0
  const __amdgpu_buffer_rsrc_t own = buffer_over_uniform(in + g.start, g.n * (int)sizeof(float));
  const int off = g.lane * (int)sizeof(float);
#pragma unroll
  for (int i = 0; i < NG; ++i) r[i] = 0u;
  for_slots<NG>(g, [&](int, int i) {
    r[i] = __builtin_amdgcn_raw_buffer_load_b32(own, off + i * 256, 0, 0);
  });
  // with a window, the raw scores on either side of a chunk: lanes 0-2 before it, lanes 3-5 after
  // its last entry (reads outside the segment return 0 and count as key 0)
  uint32_t side[kChunks];
  auto chunk_end = [&](int b) {   // entries of the wave up to the end of chunk b
    const int e = (b + 1) * kRegChunk * 64;
    return g.n < e ? g.n : e;
  };
  if (hw > 0) {
    const __amdgpu_buffer_rsrc_t all = buffer_over_uniform(in, g.L * (int)sizeof(float));
#pragma unroll
    for (int b = 0; b < kChunks; ++b) {
      side[b] = 0u;
      if (b * kRegChunk >= g.per) continue;
      const int t = g.start + (g.lane < kPoolHalo ? b * kRegChunk * 64 - kPoolHalo + g.lane
                                                  : chunk_end(b) - kPoolHalo + g.lane);
      side[b] = __builtin_amdgcn_raw_buffer_load_b32(all, t * (int)sizeof(float), 0, 0);
    }
  }
  uint32_t* c = lds.chunk[g.w];
  const uint32_t bias = hw > 0 ? kPoolBias : 0u;   // taken off again once pooled
#pragma unroll
  for (int b = 0; b < kChunks; ++b) {
    if (b * kRegChunk >= g.per) continue;
#pragma unroll
    for (int j = 0; j < kRegChunk; ++j) {
      const int i = b * kRegChunk + j;
      if (i < NG) {
        // opaque: keeps the conversion, and its wait for this load, out of the loop that issues
        // all of them
        asm volatile("" : "+v"(r[i]));
        r[i] = bits_key(r[i]) + bias;   // (with the key's last step, one instruction)
      }
    }
    if ((b + 1) * kRegChunk * 64 > g.n) {   // the chunk with the end of the wave's entries
#pragma unroll
      for (int j = 0; j < kRegChunk; ++j) {
        const int i = b * kRegChunk + j;
        if (i < NG) r[i] = i * 64 + g.lane < g.n ? r[i] : 0u;
      }
    }
    if (hw > 0) {
#pragma unroll
      for (int j = 0; j < kRegChunk; ++j)
        if (b * kRegChunk + j < NG) c[kPoolHalo + j * 64 + g.lane] = r[b * kRegChunk + j];
      // (after the slots: the end may lie inside a group)
      wave_lds_fence();
      if (g.lane < 2 * kPoolHalo && g.n > b * kRegChunk * 64) {
        const int at = g.lane < kPoolHalo ? g.lane : chunk_end(b) - b * kRegChunk * 64 + g.lane;
        const int t = g.start + b * kRegChunk * 64 - kPoolHalo + at;
        c[at] = t >= 0 && t < g.L ? bits_key(side[b]) + kPoolBias : 0u;
      }
      wave_lds_fence();
      auto pool = [&](auto half) {
#pragma unroll
        for (int j = 0; j < kRegChunk; ++j) {
          const int i = b * kRegChunk + j;
          if (i < NG) {
            const uint32_t* at = c + kPoolHalo + j * 64 + g.lane;
            uint32_t m = r[i];
#pragma unroll
            for (int d = 1; d <= decltype(half)::value; ++d) m = max(max(m, at[-d]), at[d]);
            r[i] = m - kPoolBias;
          }
        }
      };
      if (hw == 3) pool(std::integral_constant<int, 3>());   // uniform
      else if (hw == 2) pool(std::integral_constant<int, 2>());
      else pool(std::integral_constant<int, 1>());
      if ((b + 1) * kRegChunk * 64 > g.n) {
#pragma unroll
        for (int j = 0; j < kRegChunk; ++j) {
          const int i = b * kRegChunk + j;
          if (i < NG) r[i] = i * 64 + g.lane < g.n ? r[i] : 0u;
        }
      }
      wave_lds_fence();   // every lane has read before the next chunk overwrites
    }
  }
  if (pout) {
    const __amdgpu_buffer_rsrc_t dst = buffer_over_uniform(pout + g.start, g.n * (int)sizeof(float));
    for_slots<NG>(g, [&](int, int i) {   // stores past the wave's entries are dropped
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(key_value(r[i])), dst, off + i * 256, 0,
                                            0);
    });
  }
}

// Of every 64 entries this many go to the sample.
__device__ __forceinline__ int sample_share(int per) {
  const int chunks = (per + kRegChunk - 1) / kRegChunk;
  return chunks <= 1 ? 8 : (chunks <= 2 ? 4 : (chunks <= 4 ? 2 : 1));
}

// Sample of the keys (0: none) and their range into LDS.  Between two barriers of the caller (the
// first retires the pooling, whose LDS is written over).
template <int NG>
__device__ __forceinline__ void reg_sample(const RegGeom g, const uint32_t (&r)[NG], RegLds& lds) {
  const int chunks = (g.per + kRegChunk - 1) / kRegChunk, share = sample_share(g.per);
  const int used = kRegWaves * chunks * share * 8;
  if ((int)threadIdx.x >= used) lds.samp[threadIdx.x] = 0u;
  const int rows = 8 / share, col = g.lane & 7;   // one row of 8 lanes in `rows` is taken
  uint32_t mx = 0u, mn = 0xFFFFFFFFu;             // mn: smallest key but 0, minus 1
#pragma unroll
  for (int b = 0; b < (NG + kRegChunk - 1) / kRegChunk; ++b) {
    if (b * kRegChunk >= g.per) continue;
    // lane l holds the key of slot l % 8 of the chunk: a row of 8 lanes has one of each group
    uint32_t x = 0u;
#pragma unroll
    for (int j = 0; j < kRegChunk; ++j) {
      const int i = b * kRegChunk + j;
      if (i >= NG) continue;
      x = col == j ? r[i] : x;
      mx = max(mx, r[i]);
      mn = min(mn, r[i] - 1u);
    }
    // the row shifts from chunk to chunk and wave to wave
    const int rel = (g.lane / 8 - b - g.w) & 7;
    if ((rel & (rows - 1)) == 0)
      lds.samp[((g.w * chunks + b) * share + rel / rows) * 8 + col] = x;
  }
  mx = wave_max_u32(mx);
  mn = wave_max_u32(~mn);   // complement of (smallest key - 1)
  if (g.lane == 0) {
    lds.range[g.w] = mx;
    lds.range[kRegWaves + g.w] = mn;
  }
}

// Smallest and largest key of the segment (after reg_sample and a barrier).
__device__ __forceinline__ void reg_range(const RegGeom& g, const RegLds& lds, uint32_t* lo,
                                          uint32_t* hi) {
  const uint32_t v = lds.range[g.lane & (2 * kRegWaves - 1)];
  *hi = wave_max_u32((g.lane & kRegWaves) == 0 ? v : 0u);
  *lo = ~wave_max_u32((g.lane & kRegWaves) != 0 ? v : 0u) + 1u;
}

// Bracket of the k-th largest key, from the segment's smallest and largest (*lo, *hi): the k-th
// entry's expected sample rank, four standard deviations and a little to either side, which misses
// about one segment in 10,000; either end at a cell of a 1,024-cell histogram of the sample over the
// key range.  Begins after the barrier that follows reg_sample; a barrier must follow before lds.hist
// is written.
__device__ __forceinline__ void bracket_rank(const RegGeom& g, int k, RegLds& lds, uint32_t* lo,
                                             uint32_t* hi) {
  const int tid = threadIdx.x;
  const uint32_t key = lds.samp[tid];
  const uint32_t base = *lo, range = *hi - base;
  const int bits = range == 0 ? 0 : 32 - __clz(range), sh = bits > 10 ? bits - 10 : 0;
  lds.hist[tid] = 0;
  if (tid == 0) {
    lds.bracket[0] = base;   // unless some cell below holds that many samples
    lds.bracket[1] = *hi;
  }
  __syncthreads();
  if (key != 0u) atomicAdd(&lds.hist[(key - base) >> sh], 1u);
  __syncthreads();
  const float q = (float)k / (float)g.L;
  const float m = (float)k * (float)sample_share(g.per) * (1.0f / 64.0f);
  const float d = 4.0f * __builtin_sqrtf(m * (1.0f - q)) + 4.0f;
  const int above = (int)(m - d), below = (int)(m + d) + 1;
  const int cell = kCells - 1 - tid;
  const int mine = (int)lds.hist[cell];
  int64_t tot;
  const int before = (int)block_excl_scan_i64(mine, lds.scan, &tot);
  const uint32_t at = base + ((uint32_t)cell << sh), last = at + ((1u << sh) - 1u);
  if (before < below && below <= before + mine) lds.bracket[0] = at;
  if (above >= 1 && before < above && above <= before + mine && last >= at && last < *hi)
    lds.bracket[1] = last;
  __syncthreads();
  *lo = lds.bracket[0];
  *hi = lds.bracket[1];
}

// What is taken of a segment: every key above `hi` and, of the entries in [lo, hi], the first
// `need` (kRank: in the order of their keys, largest first, then of their index; kIndex: all one
// key, in the order of their index; kNone: none).
struct RegCut {
  uint32_t lo, hi;
  uint64_t need;
  enum Mode { kNone, kRank, kIndex } mode;
};

// The cut that keeps the k largest entries (0 < k < L), given a bracket.  Ends with a barrier.
// lo is at least 1 (reg_range leaves key 0 out), so that neither the counts nor the list below hold a
// slot without an entry.
template <int NG>
__device__ __forceinline__ RegCut cut_rank(const RegGeom& g, int k, const uint32_t (&r)[NG],
                                           RegLds& lds, uint32_t lo, uint32_t hi) {
  const int tid = threadIdx.x;
  uint32_t need = 0;      // of the entries in [lo, hi], once `counted`
  bool counted = false;   // the entries above hi are accounted for in need
  bool whole = false;     // [lo, hi] is the segment's whole range
#pragma unroll 1
  for (;;) {
    lds.hist[tid] = 0;
    __syncthreads();
    const uint32_t range = hi - lo;
    const int bits = range == 0 ? 0 : 32 - __clz(range), sh = bits > 10 ? bits - 10 : 0;
    uint32_t above = 0;   // wave-uniform
    for_slots<NG>(g, [&](int, int i) {
      above += __popcll(__ballot(r[i] > hi));
      const uint32_t d = r[i] - lo;   // keys below lo wrap to above the range
      if (d <= range) atomicAdd(&lds.hist[d >> sh], 1u);
    });
    __syncthreads();
    const int bin = kCells - 1 - tid;
    const uint32_t mine = lds.hist[bin];
    int64_t tot;
    const int64_t ex = block_excl_scan_i64(
        ((int64_t)(g.lane == 0 ? above : 0u) << 32) + mine, lds.scan, &tot);
    if (!counted) {
      const int rest = k - (int)(tot >> 32);
      if (rest < 0 || (uint32_t)rest > (uint32_t)tot) {   // the bracket missed: the whole range
        // every key but 0 is taken, and of those of key 0 (NaNs) the first by their index
        if (whole) return RegCut{0u, 0u, (uint64_t)(rest - (int)(uint32_t)tot), RegCut::kIndex};
        reg_range(g, lds, &lo, &hi);
        whole = true;
        continue;
      }
      if (rest == 0) return RegCut{lo, hi, 0, RegCut::kNone};
      need = (uint32_t)rest;
      counted = true;
    }
    const uint32_t before = (uint32_t)ex;
    if (before < need && need <= before + mine) {   // one thread
      lds.bin = bin;
      lds.bin_need = need - before;
      lds.bin_count = mine;
    }
    if (tid == 0) lds.listed = 0;
    __syncthreads();
    const uint32_t cell = lo + ((uint32_t)lds.bin << sh), width = (1u << sh) - 1u;
    const uint32_t count = lds.bin_count;
    need = (uint32_t)lds.bin_need;
    hi = width > hi - cell ? hi : cell + width;
    lo = cell;
    if (count == need)   // the whole bin is kept: every key from its lowest (at least 1) up
      return RegCut{lo, lo - 1u, 0, RegCut::kNone};
    if (count <= (uint32_t)kListMax) return RegCut{lo, hi, need, RegCut::kRank};
    if (sh == 0) return RegCut{lo, lo, need, RegCut::kIndex};
    __syncthreads();   // lds.bin and its fellows are read before they are written again
  }
}

// What a cut takes, as the last entry in the order (key descending, then index ascending): every
// key above `key`, and those equal to it up to index `at`.
struct RegLast {
  uint32_t key;
  int32_t at;
};

// How many slots hold `key`.
template <int NG>
__device__ __forceinline__ uint32_t count_key(const RegGeom& g, uint32_t key,
                                              const uint32_t (&r)[NG], RegLds& lds) {
  uint32_t same = 0;   // wave-uniform
  for_slots<NG>(g, [&](int, int i) { same += __popcll(__ballot(r[i] == key)); });
  int64_t tot;
  block_excl_scan_i64(g.lane == 0 ? same : 0u, lds.scan, &tot);
  return (uint32_t)tot;
}

// The cut where every entry has the key `key`, or key 0 (0 < k < L).  Put into the bins such a segment
// would take an LDS atomic on one bin per entry: 55 us against 27 for 4 segments of 35,000 zeros.
template <int NG>
__device__ __forceinline__ RegCut cut_equal(const RegGeom& g, uint32_t key, int k,
                                            const uint32_t (&r)[NG], RegLds& lds) {
  const uint32_t same = key != 0u ? count_key(g, key, r, lds) : 0u;
  return (uint32_t)k <= same ? RegCut{key, key, (uint64_t)k, RegCut::kIndex}
                             : RegCut{0u, 0u, (uint64_t)((uint32_t)k - same), RegCut::kIndex};
}

// The last of the first `want` entries equal to `key`, in index order (1 <= want; all of them if
// there are fewer).  Ends with a barrier.
template <int NG>
__device__ __forceinline__ RegLast index_last(const RegGeom& g, uint32_t key, uint64_t want,
                                              const uint32_t (&r)[NG], RegLds& lds) {
  uint32_t in_lo = 0, in_hi = 0;
  for_slots<NG>(g, [&](int, int i) {
    const uint64_t in = __ballot(r[i] == key);
    in_lo = llvm_writelane((uint32_t)in, i, in_lo);
    in_hi = llvm_writelane((uint32_t)(in >> 32), i, in_hi);
  });
  uint64_t in = (((uint64_t)in_hi << 32) | in_lo) & reg_real(g);
  int64_t tot;
  const uint64_t before = (uint64_t)block_excl_scan_i64(__popcll(in), lds.scan, &tot);
  if (want > (uint64_t)tot) return RegLast{key, g.L};
  if (before < want && want <= before + __popcll(in)) {
    for (uint64_t skip = want - before - 1; skip; --skip) in &= in - 1;
    lds.last_at = g.start + g.lane * 64 + __builtin_ctzll(in);
  }
  __syncthreads();
  return RegLast{key, lds.last_at};
}

// Lists the entries with keys in [lo, hi] (lds.listed is 0 and visible).  Returns how many there
// are; no more than kListMax of them are in the list.  Ends with a barrier.
template <int NG>
__device__ __forceinline__ int list_entries(const RegGeom& g, uint32_t lo, uint32_t hi,
                                            const uint32_t (&r)[NG], RegLds& lds) {
  const uint32_t width = hi - lo;
  int first = g.first();
  asm volatile("" : "+v"(first));   // opaque: no slot's index is kept from one call for the next
  for_slots<NG>(g, [&](int, int i) {
    if (r[i] - lo <= width) {
      const int at = atomicAdd(&lds.listed, 1);
      if (at < kListMax) {
        lds.list_key[at] = r[i];
        lds.list_at[at] = first + i * 64;
      }
    }
  });
  __syncthreads();
  return lds.listed;
}

// The last of the n <= kListMax listed entries taken, in the order (key descending, then index
// ascending), when their weights are to reach `need` (1 <= need <= their sum).  weight(key): 1 for
// a selection, the entry's mass for the top-p set.  Ends with a barrier.
template <typename Weight>
__device__ __forceinline__ RegLast rank_last(const RegGeom& g, int n, uint64_t need, RegLds& lds,
                                             Weight weight) {
  static_assert(kListMax <= 64, "an entry per lane");
  if (g.w == 0) {
    const uint32_t key = g.lane < n ? lds.list_key[g.lane] : 0u;
    const int at = g.lane < n ? lds.list_at[g.lane] : 0;
    uint64_t before = 0;
    for (int c = 0; c < n; ++c) {
      const uint32_t kc = (uint32_t)__builtin_amdgcn_readlane((int)key, c);
      const int ac = __builtin_amdgcn_readlane(at, c);
      if (kc > key || (kc == key && ac < at)) before += weight(kc);
    }
    if (g.lane < n && before < need && need <= before + weight(key)) {
      lds.last_key = key;
      lds.last_at = at;
    }
  }
  __syncthreads();
  return RegLast{lds.last_key, lds.last_at};
}

// The last entry that a cut takes.
template <int NG>
__device__ __forceinline__ RegLast cut_last(const RegGeom& g, const RegCut cut,
                                            const uint32_t (&r)[NG], RegLds& lds) {
  if (cut.mode == RegCut::kNone) return RegLast{cut.hi, -1};
  if (cut.mode == RegCut::kIndex) return index_last(g, cut.lo, cut.need, r, lds);
  const int n = list_entries(g, cut.lo, cut.hi, r, lds);
  return rank_last(g, n, cut.need, lds, [](uint32_t) { return (uint64_t)1; });
}

// The entries up to the last one, as one mask per group: lane i of a wave gets the mask of the
// wave's slot i.
template <int NG>
__device__ __forceinline__ uint64_t take_masks(const RegGeom& g, const RegLast last,
                                               const uint32_t (&r)[NG]) {
  const uint32_t last_key = (uint32_t)__builtin_amdgcn_readfirstlane((int)last.key);
  const int last_slot_at = __builtin_amdgcn_readfirstlane(last.at) - g.start;   // in this wave
  uint32_t gt_lo = 0, gt_hi = 0, eq_lo = 0, eq_hi = 0;
  for_slots<NG>(g, [&](int, int i) {
    const uint64_t gt = __ballot(r[i] > last_key), eq = __ballot(r[i] == last_key);
    gt_lo = llvm_writelane((uint32_t)gt, i, gt_lo);
    gt_hi = llvm_writelane((uint32_t)(gt >> 32), i, gt_hi);
    eq_lo = llvm_writelane((uint32_t)eq, i, eq_lo);
    eq_hi = llvm_writelane((uint32_t)(eq >> 32), i, eq_hi);
  });
  const int upto = last_slot_at - g.lane * 64;   // the last index within this lane's group
  const uint64_t some = upto < 0 ? 0ull : (upto >= 63 ? ~0ull : (2ull << upto) - 1ull);
  return ((((uint64_t)gt_hi << 32) | gt_lo) | ((((uint64_t)eq_hi << 32) | eq_lo) & some)) &
         reg_real(g);
}

// Kept entries in ascending order: put(j, t, key) for the j-th of them, entry t.  `keep`: the
// masks of take_masks.
template <int NG, typename Put>
__device__ __forceinline__ void emit_masks(const RegGeom& g, uint64_t keep,
                                           const uint32_t (&r)[NG], RegLds& lds, Put put) {
  int64_t tot;
  const int pos = (int)block_excl_scan_i64(__popcll(keep), lds.scan, &tot);
  const uint32_t k_lo = (uint32_t)keep, k_hi = (uint32_t)(keep >> 32);
  for_slots<NG>(g, [&](int, int i) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)k_lo, i);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)k_hi, i);
    const int p = __builtin_amdgcn_readlane(pos, i);
    if (__builtin_amdgcn_inverse_ballot_w64(((uint64_t)hi << 32) | lo))
      put(p + (int)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u)),
          g.first() + i * 64, r[i]);
  });
}

// The k largest of the keys in registers (ties to the lower index) in ascending index order:
// put(j, t, key).  The LDS is free on entry and on exit.
template <int NG, typename Put>
__device__ __forceinline__ void reg_topk(const RegGeom& g, int k, const uint32_t (&r)[NG],
                                         RegLds& lds, Put put) {
  if (k <= 0) return;
  uint64_t keep;
  __syncthreads();   // the pooling's LDS has been read
  if (k < g.L) {
    reg_sample(g, r, lds);
    __syncthreads();
    uint32_t lo, hi;
    reg_range(g, lds, &lo, &hi);
    RegCut cut;
    if (lo == hi) {
      cut = cut_equal(g, lo, k, r, lds);
    } else {
      bracket_rank(g, k, lds, &lo, &hi);
      cut = cut_rank(g, k, r, lds, lo, hi);
    }
    keep = take_masks(g, cut_last(g, cut, r, lds), r);
  } else {   // everything
    keep = reg_real(g);
  }
  emit_masks(g, keep, r, lds, put);
}

// ---- the top-p hit set -------------------------------------------------------------------
// floor(v * 2^S) for the positive float whose order key is `key` (0 for v <= 0), by integer
// shifts of the significand: exact, as long as the result stays below 2^64.
__device__ __forceinline__ uint64_t fixed_mass(uint32_t key, int S) {
  if (key <= 0x80000000u) return 0ull;   // negative or zero
  const uint32_t u = key & 0x7FFFFFFFu, ex = u >> 23;
  const uint64_t sig = (u & 0x7FFFFFu) | (ex ? 0x800000u : 0u);
  const int sh = (ex ? (int)ex : 1) - 150 + S;   // v = sig * 2^((ex ? ex : 1) - 150)
  return sh >= 0 ? sig << sh : (sh > -64 ? sig >> -sh : 0ull);
}

// The same by float operations that are exact here: v * 2^(S - 32) below 2^32, its integer part,
// and 2^32 times the rest truncated (half the instructions, and none on 64 bits; where the first
// product loses bits to underflow the mass is 0 either way).
__device__ __forceinline__ uint64_t fixed_mass_below32(uint32_t key, int S) {
  const float x = fmaxf(__builtin_amdgcn_ldexpf(__uint_as_float(key ^ 0x80000000u), S - 32), 0.0f);
  const uint32_t hi = (uint32_t)x;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_ldexpf(__builtin_amdgcn_fractf(x), 32);
  return ((uint64_t)hi << 32) | lo;
}

// Bracket of the key at which the mass, largest keys first, reaches the share p (0 < p < 1) of the
// total, from the masses of the sample (all_hi: the largest key, positive): four standard
// deviations of the sample's mass above that key to either side.  LDS as for bracket_rank.
__device__ __forceinline__ void bracket_mass(const RegGeom& g, float p, RegLds& lds,
                                             uint32_t all_lo, uint32_t all_hi, uint32_t* lo,
                                             uint32_t* hi) {
  const int tid = threadIdx.x;
  constexpr uint32_t kLeast = 0x80000001u;   // key of the smallest positive float
  const uint32_t key = lds.samp[tid];
  const uint32_t base = all_lo < kLeast ? kLeast : all_lo, range = all_hi - base;
  const int bits = range == 0 ? 0 : 32 - __clz(range), sh = bits > 10 ? bits - 10 : 0;
  lds.mass[tid] = 0;
  if (tid == 0) {
    lds.bracket[0] = base;
    lds.bracket[1] = all_hi;
    lds.cut_value = 1.0f;
  }
  __syncthreads();
  // masses and their squares relative to the largest entry's, 2^21 and 2^20 to the unit, in the
  // halves of a word: neither sum over the sample reaches 2^32
  const float unit = 1.0f / key_value(all_hi);
  if (key >= base) {
    const float x = key_value(key) * unit;
    atomicAdd((unsigned long long*)&lds.mass[(key - base) >> sh],
              ((unsigned long long)(uint32_t)(x * 2097152.0f) << 32) +
                  (uint32_t)(x * x * 1048576.0f));
  }
  __syncthreads();
  const int cell = kCells - 1 - tid;
  const uint64_t mine = lds.mass[cell];
  int64_t tot;
  const uint64_t ex = (uint64_t)block_excl_scan_i64((int64_t)mine, lds.scan, &tot);
  const float before = (float)(ex >> 32), after = (float)((ex + mine) >> 32);
  const float all = (float)((uint64_t)tot >> 32), squares = 2.0f * (float)(uint32_t)tot;
  const uint32_t at = base + ((uint32_t)cell << sh), last = at + ((1u << sh) - 1u);
  const float want = p * all;
  if (before < want && want <= after) lds.cut_value = key_value(at) * unit;
  __syncthreads();
  // variance of (mass of the sample above the key) - p * (mass of the sample), in units of 2^-42:
  // entries above count (1 - p) of their mass, those below, none larger than the key's value, p
  const float value = lds.cut_value * 2097152.0f, rest = 1.0f - p;
  const float d = 4.0f * __builtin_sqrtf(p * p * rest * all * value +
                                         rest * rest * squares * 2097152.0f) + 4.0f * value;
  const float above = want - d, below = want + d;
  if (before < below && below <= after) lds.bracket[0] = at;
  if (above > 0.0f && before < above && above <= after && last >= at && last < all_hi)
    lds.bracket[1] = last;
  __syncthreads();
  *lo = lds.bracket[0];
  *hi = lds.bracket[1];
}

// The hit entries (see the top-p section of select.hip) as one mask per group.  The LDS is free on
// entry and on exit.
template <int NG>
__device__ __forceinline__ uint64_t reg_topp(const RegGeom& g, float top_p,
                                             const uint32_t (&r)[NG], RegLds& lds) {
  const int tid = threadIdx.x;
  constexpr uint32_t kZero = 0x80000000u;   // order key of 0
  __syncthreads();
  reg_sample(g, r, lds);
  __syncthreads();
  uint32_t all_lo, all_hi, lo, hi;
  reg_range(g, lds, &all_lo, &all_hi);
  const float vmax = key_value(all_hi);
  if (!(vmax > 0.f) || !(top_p > 0.f)) return 0ull;          // no positive mass to reach
  if (top_p >= 1.f) return take_masks(g, RegLast{kZero, -1}, r);   // every positive score
  int e;
  frexpf(vmax, &e);   // every score < 2^e
  const int lg = 32 - __clz((uint32_t)g.L + 1u);   // L + 1 <= 2^lg
  const int S = 62 - e - lg;                       // total < L * 2^(e + S) < 2^62
  auto mass_of = [&](uint32_t key) { return fixed_mass_below32(key, S); };   // < 2^(62 - lg)
  if (all_lo == all_hi) {   // equal scores: the first ceil(target / mass) of them, without the bins
    const uint64_t m = mass_of(all_hi), all = m * count_key(g, all_hi, r, lds);
    const uint64_t target = (uint64_t)ceil((double)top_p * (double)all);   // > 0
    return take_masks(g, index_last(g, all_hi, (target + m - 1) / m, r, lds), r);
  }
  bracket_mass(g, top_p, lds, all_lo, all_hi, &lo, &hi);
  uint64_t need = 0;      // of the mass in [lo, hi], once `counted`
  bool counted = false, whole = false;
#pragma unroll 1
  for (;;) {
    lds.mass[tid] = 0;
    if (tid == 0) lds.listed = 0;
    __syncthreads();
    const uint32_t range = hi - lo;
    const int bits = range == 0 ? 0 : 32 - __clz(range), sh = bits > 10 ? bits - 10 : 0;
    uint64_t all = 0, above = 0;
    // (opaque keys and masses: nothing computed from a slot is kept for the next pass, and the
    // sums run slot by slot)
    auto add_up = [&](auto first) {
      for_slots<NG>(g, [&](int, int i) {
        uint32_t kk = r[i];
        asm volatile("" : "+v"(kk));
        const uint32_t d = kk - lo;
        if constexpr (decltype(first)::value) {
          uint64_t m = mass_of(kk);
          asm volatile("" : "+v"(m));
          all += m;
          above += kk > hi ? m : 0ull;
          if (d <= range) atomicAdd((unsigned long long*)&lds.mass[d >> sh], (unsigned long long)m);
        } else if (d <= range) {
          atomicAdd((unsigned long long*)&lds.mass[d >> sh], (unsigned long long)mass_of(kk));
        }
      });
    };
    if (counted) add_up(std::false_type());
    else add_up(std::true_type());
    if (!counted) {
      all = (uint64_t)wave_incl_scan_i64((int64_t)all);
      above = (uint64_t)wave_incl_scan_i64((int64_t)above);
      if (g.lane == 63) {
        lds.sum[g.w] = all;
        lds.sum[kRegWaves + g.w] = above;
      }
    }
    __syncthreads();
    const int bin = kCells - 1 - tid;
    const uint64_t mine = lds.mass[bin];
    int64_t tot;
    const uint64_t before = (uint64_t)block_excl_scan_i64((int64_t)mine, lds.scan, &tot);
    if (!counted) {
      all = above = 0;
#pragma unroll
      for (int u = 0; u < kRegWaves; ++u) {
        all += lds.sum[u];
        above += lds.sum[kRegWaves + u];
      }
      const double want = ceil((double)top_p * (double)all);
      const uint64_t target = want > 0.0 ? (uint64_t)want : 0ull;
      if (target == 0) return 0ull;
      if (target <= above || target - above > (uint64_t)tot) {   // the bracket missed
        if (whole) return 0ull;   // not with finite scores
        lo = all_lo <= kZero ? kZero + 1u : all_lo;
        hi = all_hi;
        whole = true;
        __syncthreads();   // lds.sum has been read
        continue;
      }
      need = target - above;
      counted = true;
    }
    if (before < need && need <= before + mine) {   // one thread
      lds.bin = bin;
      lds.bin_need = need - before;
    }
    __syncthreads();
    const uint32_t cell = lo + ((uint32_t)lds.bin << sh), width = (1u << sh) - 1u;
    need = lds.bin_need;
    hi = width > hi - cell ? hi : cell + width;
    lo = cell;
    const int n = list_entries(g, lo, hi, r, lds);
    RegLast last;
    if (n <= kListMax) {
      last = rank_last(g, n, need, lds, mass_of);
    } else if (sh == 0) {   // one key: the first ceil(need / mass) of its entries
      const uint64_t m = mass_of(lo);
      last = index_last(g, lo, m == 0 ? ~0ull : (need + m - 1) / m, r, lds);
    } else {
      __syncthreads();   // lds.listed and lds.bin have been read
      continue;
    }
    return take_masks(g, last, r);
  }
}

// KS' = decay * KS + (hit ? score : 0), each operation rounded to fp32, to ks in place; the keys of
// the pooled scores in r become those of KS'; hit flags to hit_out when given.
template <int NG>
__device__ __forceinline__ void reg_keep_scores(const RegGeom& g, float decay, uint64_t hits,
                                                float* ks, uint8_t* hit_out, uint32_t (&r)[NG]) {
  constexpr int kChunks = (NG + kRegChunk - 1) / kRegChunk;
  const __amdgpu_buffer_rsrc_t rk = buffer_over_uniform(ks + g.start, g.n * (int)sizeof(float));
  const __amdgpu_buffer_rsrc_t rh = buffer_over_uniform(hit_out + g.start, hit_out ? g.n : 0);
  const int off = g.lane * (int)sizeof(float);
  const uint32_t h_lo = (uint32_t)hits, h_hi = (uint32_t)(hits >> 32);
  uint32_t next[kRegChunk];   // the next chunk's keep scores, in flight
  auto fetch = [&](int b) {
#pragma unroll
    for (int j = 0; j < kRegChunk; ++j)
      next[j] = __builtin_amdgcn_raw_buffer_load_b32(rk, off + (b * kRegChunk + j) * 256, 0, 0);
  };
  fetch(0);
#pragma unroll
  for (int b = 0; b < kChunks; ++b) {
    if (b * kRegChunk >= g.per) continue;
    uint32_t old[kRegChunk];
#pragma unroll
    for (int j = 0; j < kRegChunk; ++j) old[j] = next[j];
    if (b + 1 < kChunks) fetch(b + 1);   // (reads past the wave's entries return 0)
#pragma unroll
    for (int j = 0; j < kRegChunk; ++j) {
      const int i = b * kRegChunk + j;
      if (i >= NG) continue;
      const uint64_t m = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)h_hi, i) << 32) |
                         (uint32_t)__builtin_amdgcn_readlane((int)h_lo, i);
      const bool hit = __builtin_amdgcn_inverse_ballot_w64(m);
      const float c = hit ? key_value(r[i]) : 0.0f;
      const uint32_t nk = __float_as_uint(__fadd_rn(__fmul_rn(decay, __uint_as_float(old[j])), c));
      __builtin_amdgcn_raw_buffer_store_b32(nk, rk, off + i * 256, 0, 0);
      if (hit_out)
        __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(hit ? 1 : 0), rh, g.lane + i * 64, 0, 0);
      r[i] = bits_key(nk);
    }
    if ((b + 1) * kRegChunk * 64 > g.n) {   // the chunk with the end of the wave's entries
#pragma unroll
      for (int j = 0; j < kRegChunk; ++j) {
        const int i = b * kRegChunk + j;
        if (i < NG) r[i] = i * 64 + g.lane < g.n ? r[i] : 0u;
      }
    }
  }
}
