// Per-unit stable ordering of keys by score, descending, ties by position.
//
// One workgroup (16 waves) sorts one unit's segment with a least-significant-
// digit radix sort: 4 passes of 8-bit digits over the order-inverting key
// transform of the fp32 score (desc_key).  One counting pass first forms all
// four digit histograms with LDS atomics (and the fp64 sum of (s)_+, the
// normalizer of a_j).
// Each pass then walks the segment in tiles of 16 * 64 * R elements; wave w
// holds the R rounds of 64 consecutive elements at offset 64 R w:
//   rank     lanes with equal digits are found with 8 ballots; an element's
//            rank among equal digits of its wave is a per-wave LDS counter
//            plus mbcnt within the round (input order);
//   offsets  per digit, an exclusive scan over the waves, and per tile an
//            exclusive scan over the digits of the tile's digit counts (the
//            two run concurrently on different waves);
//   stage    every element is written to LDS at its digit-major position in
//            the tile (stable);
//   write    thread i stores staged element i to the digit's running bucket
//            offset plus its position inside the tile's run of that digit,
//            so consecutive threads write consecutive addresses.
// Ranking in input order and runs in tile order make every pass stable, so
// equal scores keep ascending position.  The next tile's elements are loaded
// while the current one is ranked.
//
// That is a serial chain of tiles, which leaves most of the chip idle with few
// units.  So most units of more than kSortRun elements are cut by value into
// buckets of about half of it, each sorted by a workgroup of its own, entirely in
// LDS (units of up to kSortRun by one workgroup, without buckets):
//   splitters  one workgroup per unit sorts kSortOver samples per bucket,
//              one from each of as many equal stretches of positions, and
//              picks every kSortOver-th;
//   count      one workgroup per tile of kSortRun elements: each element's
//              bucket (a search among the splitters) and the tile's counts;
//   scatter    one per tile: elements to their buckets, in position order;
//   buckets    one per bucket: its elements in order, to their final ranks.
// Splitters and elements compare by (key, position), so ties spread over the
// buckets like distinct keys.  A bucket beyond kSortRun elements (twice its
// expected size: samples that misjudge the keys) is sorted by its
// workgroup through memory instead.  Four launches, each element read three
// times and written twice.  sort_buckets() in api.hip holds the rule.
#include <type_traits>

#include "stages.h"

namespace certkv {

constexpr int kSortThreads = 1024;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortRounds = 8;
constexpr int kSortTile = kSortThreads * kSortRounds;  // 8192 elements

// Lanes of the wave whose 8-bit digit equals this lane's (among `valid`).
// Per bit, the lanes agreeing with this lane are the ballot of the bit when
// it is set here and its complement when it is clear: ballot ^ m with m the
// bit sign-extended from ~digit (0 or all ones), which keeps the selection a
// per-lane xor of a wave-uniform mask.
__device__ __forceinline__ uint64_t match_digit(uint32_t digit, bool valid) {
  const uint64_t v = __ballot(valid);
  uint32_t plo = (uint32_t)v, phi = (uint32_t)(v >> 32);
  const uint32_t nd = ~digit;
#pragma unroll
  for (int bit = 0; bit < 8; ++bit) {
    const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)nd, bit, 1);
    const uint64_t bb = __ballot(m == 0u);
    plo &= (uint32_t)bb ^ m;
    phi &= (uint32_t)(bb >> 32) ^ m;
  }
  return ((uint64_t)phi << 32) | plo;
}

__device__ __forceinline__ uint32_t count_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Exclusive scan of 256 counters by one wave (4 per lane), in place.
__device__ __forceinline__ void wave_scan256(uint32_t* v, int lane) {
  uint32_t c[4], run = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    c[j] = v[lane * 4 + j];
    run += c[j];
  }
  uint32_t incl = run;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(incl, off, 64);
    if (lane >= off) incl += y;
  }
  uint32_t excl = incl - run;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    v[lane * 4 + j] = excl;
    excl += c[j];
  }
}

__global__ __launch_bounds__(kSortThreads) void seg_sort_kernel(
    Geo g, SeqTab st, const float* __restrict__ scores, uint32_t* __restrict__ keysA,
    int32_t* __restrict__ valsA, uint32_t* __restrict__ keysB, int32_t* __restrict__ valsB,
    uint32_t* __restrict__ keys_out, int32_t* __restrict__ perm_out,
    double* __restrict__ ssum_out) {
  __shared__ uint32_t hist[4][256];
  __shared__ uint32_t bucket[256];      // running start of each digit's bucket
  __shared__ uint32_t tile_tot[2][256]; // digit counts of the tile, by tile parity
  __shared__ uint32_t tile_start[256];  // digit-major start inside the tile
  __shared__ uint32_t wave_cnt[kSortWaves][256];
  __shared__ uint32_t stage_key[kSortTile];
  __shared__ int32_t stage_val[kSortTile];
  __shared__ double dred[kSortWaves];

  const int h = blockIdx.x % g.H;
  const int bl = blockIdx.x / g.H;
  const int l = blockIdx.y;
  if (bl >= st.count) return;
  const int b = st.first + bl;
  const int n = st.len[bl];
  const int64_t base = lht_base(g, l, h, st.start[bl]);
  const int64_t u = unit_index(g, l, b, h);
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  // positions from wkeep on are the kept window: key 0 ranks them first
  const int wkeep = n - g.keep_w;

  for (int i = threadIdx.x; i < 4 * 256; i += kSortThreads) (&hist[0][0])[i] = 0u;
  for (int i = threadIdx.x; i < 2 * 256; i += kSortThreads) (&tile_tot[0][0])[i] = 0u;
  __syncthreads();

  // Counting pass: four digit histograms and the fp64 sum of (s)_+.  The
  // next tile's scores are loaded while the current one is counted.
  {
    double psum = 0.0;
    auto load_scores = [&](int t0, float (&x)[kSortRounds]) {
#pragma unroll
      for (int r = 0; r < kSortRounds; ++r) {
        const int e = t0 + wave * 64 * kSortRounds + r * 64 + lane;
        const float v = scores[base + min(e, n - 1)];  // clamped: no branch around the load
        x[r] = e < n ? v : 0.f;
      }
    };
    float sv[kSortRounds], sn[kSortRounds];
    load_scores(0, sv);
    for (int t0 = 0; t0 < n; t0 += kSortTile) {
      load_scores(t0 + kSortTile, sn);  // unconditional: clamped reads, no branch
#pragma unroll
      for (int r = 0; r < kSortRounds; ++r) {
        const int e = t0 + wave * 64 * kSortRounds + r * 64 + lane;
        const bool valid = e < n;
        if (valid && sv[r] > 0.f) psum += (double)sv[r];
        const uint32_t key = e >= wkeep ? 0u : desc_key(sv[r]);
        if (valid) {
#pragma unroll
          for (int p = 0; p < 3; ++p) atomicAdd(&hist[p][(key >> (8 * p)) & 255u], 1u);
        }
        // The top digit holds the score's sign and upper exponent bits, so a
        // wave sees few distinct values: one atomic per distinct digit
        // instead of one per lane on a handful of addresses.
        const uint32_t d3 = key >> 24;
        uint64_t todo = __ballot(valid);
        while (todo) {
          const int leader = __builtin_ctzll(todo);
          const uint32_t dl = __builtin_amdgcn_readlane(d3, leader);
          const uint64_t same = __ballot(d3 == dl) & todo;
          if (lane == leader) atomicAdd(&hist[3][dl], (uint32_t)__popcll(same));
          todo &= ~same;
        }
      }
#pragma unroll
      for (int r = 0; r < kSortRounds; ++r) sv[r] = sn[r];
    }
    psum = wave_sum(psum);
    if (lane == 0) dred[wave] = psum;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double tot = 0.0;
    for (int w = 0; w < kSortWaves; ++w) tot += dred[w];
    ssum_out[u] = tot;
  }

  // One pass per digit, instantiated per pass so that its input (the scores
  // or the previous pass's output) is fixed at compile time and no branch
  // splits the tile loads.
  auto pass = [&](auto pass_tag) {
    constexpr int p = decltype(pass_tag)::value;
    const uint32_t* kin = p == 1 || p == 3 ? keysB : keysA;
    const int32_t* vin = p == 1 || p == 3 ? valsB : valsA;
    uint32_t* kout = (p == 0 || p == 2) ? keysB : (p == 1 ? keysA : keys_out);
    int32_t* vout = (p == 0 || p == 2) ? valsB : (p == 1 ? valsA : perm_out);
    const int sh = 8 * p;
    if (wave == 0) {
      for (int j = 0; j < 4; ++j) bucket[lane * 4 + j] = hist[p][lane * 4 + j];
      wave_scan256(bucket, lane);
    }
    // Loads through range-checked buffers: elements at or beyond n read as
    // zero, so no clamp or branch sits around them.  The first pass loads
    // the raw score bits and forms their radix keys (and the kept window's
    // zero keys) only when the tile is ranked, so that the next tile's loads
    // stay in flight meanwhile.
    const BufRsrc kin_r = make_rsrc(p == 0 ? (const void*)(scores + base) : (const void*)(kin + base),
                                    (uint32_t)n * 4u);
    const BufRsrc vin_r = make_rsrc(vin + base, (uint32_t)n * 4u);
    const BufRsrc kout_r = make_rsrc(kout + base, (uint32_t)n * 4u);
    const BufRsrc vout_r = make_rsrc(vout + base, (uint32_t)n * 4u);
    auto load = [&](int t0, uint32_t (&key)[kSortRounds], int32_t (&val)[kSortRounds]) {
#pragma unroll
      for (int r = 0; r < kSortRounds; ++r) {
        const int e = t0 + wave * 64 * kSortRounds + r * 64 + lane;
        const uint32_t off = (uint32_t)e * 4u;
        if (p == 0) {
          key[r] = buf_load_u32(kin_r, off);
          val[r] = e;
        } else {
          key[r] = buf_load_u32(kin_r, off);
          val[r] = (int32_t)buf_load_u32(vin_r, off);
        }
      }
    };
    uint32_t key[kSortRounds], nkey[kSortRounds];
    int32_t val[kSortRounds], nval[kSortRounds];
    load(0, key, val);
    for (int t0 = 0; t0 < n; t0 += kSortTile) {
      const int tp = (t0 / kSortTile) & 1;  // tile parity
#pragma unroll
      for (int j = 0; j < 4; ++j) wave_cnt[wave][lane * 4 + j] = 0u;
      // prefetch, unconditionally (past the end the range check reads zeros),
      // so that no branch makes the compiler wait for it before the ranking
      load(t0 + kSortTile, nkey, nval);
      if (p == 0) {
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
          const int e = t0 + wave * 64 * kSortRounds + r * 64 + lane;
          key[r] = e >= wkeep ? 0u : desc_key(__uint_as_float(key[r]));
        }
      }
      // rank within the wave
      uint32_t rank[kSortRounds];
#pragma unroll
      for (int r = 0; r < kSortRounds; ++r) {
        const int e = t0 + wave * 64 * kSortRounds + r * 64 + lane;
        const bool ok = e < n;
        const uint32_t dg = (key[r] >> sh) & 255u;
        const uint64_t peers = match_digit(dg, ok);
        const uint32_t below = count_below(peers);
        uint32_t pre = 0;
        if (ok) pre = wave_cnt[wave][dg];
        rank[r] = pre + below;
        if (ok && below == 0) {
          const uint32_t c = (uint32_t)__popcll(peers);
          wave_cnt[wave][dg] = pre + c;
          atomicAdd(&tile_tot[tp][dg], c);
        }
      }
      __syncthreads();
      // per digit: exclusive scan over the waves (waves 1-4), over the digits
      // of the tile counts (wave 0) and the previous tile's advance of the
      // bucket offsets (waves 5-8; every wave is past that tile's writes),
      // concurrently.  The previous tile's counts are cleared for the tile
      // after this one.
      if (wave == 0) {
        for (int j = 0; j < 4; ++j) tile_start[lane * 4 + j] = tile_tot[tp][lane * 4 + j];
        wave_scan256(tile_start, lane);
      } else if (threadIdx.x >= 320 && threadIdx.x < 320 + 256) {
        const int d = threadIdx.x - 320;
        if (t0 > 0) bucket[d] += tile_tot[tp ^ 1][d];
        tile_tot[tp ^ 1][d] = 0u;
      } else if (threadIdx.x < 256 + 64) {
        const int d = threadIdx.x - 64;
        uint32_t c[kSortWaves];
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) c[w] = wave_cnt[w][d];  // all reads in flight
        uint32_t run = 0;
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) {
          wave_cnt[w][d] = run;
          run += c[w];
        }
      }
      __syncthreads();
      // stage in digit-major order
#pragma unroll
      for (int r = 0; r < kSortRounds; ++r) {
        const int e = t0 + wave * 64 * kSortRounds + r * 64 + lane;
        if (e < n) {
          const uint32_t dg = (key[r] >> sh) & 255u;
          const uint32_t lp = tile_start[dg] + wave_cnt[wave][dg] + rank[r];
          stage_key[lp] = key[r];
          stage_val[lp] = val[r];
        }
      }
      __syncthreads();
      // coalesced write of the staged tile
      const int cnt = min(kSortTile, n - t0);
      {
        uint32_t kk[kSortRounds], dst[kSortRounds];
        int32_t vv[kSortRounds];
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
          const int i = threadIdx.x + r * kSortThreads;
          kk[r] = i < cnt ? stage_key[i] : 0u;
          vv[r] = i < cnt ? stage_val[i] : 0;
        }
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
          const int i = threadIdx.x + r * kSortThreads;
          const uint32_t d = (kk[r] >> sh) & 255u;
          dst[r] = bucket[d] + (uint32_t)i - tile_start[d];
        }
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
          const int i = threadIdx.x + r * kSortThreads;
          if (i < cnt) {
            buf_store_u32(kout_r, dst[r] * 4u, kk[r]);
            buf_store_u32(vout_r, dst[r] * 4u, (uint32_t)vv[r]);
          }
        }
      }
#pragma unroll
      for (int r = 0; r < kSortRounds; ++r) {
        key[r] = nkey[r];
        val[r] = nval[r];
      }
    }
    // the last tile's counts (the other parity is already clear)
    if (threadIdx.x < 256) tile_tot[((n - 1) / kSortTile) & 1][threadIdx.x] = 0u;
    __syncthreads();  // the pass's output is the next pass's input
  };
  pass(std::integral_constant<int, 0>());
  pass(std::integral_constant<int, 1>());
  pass(std::integral_constant<int, 2>());
  pass(std::integral_constant<int, 3>());
  // Kept window: its keys sorted as 0 (ahead of every score) and so hold
  // ranks 0..w-1 in position order; give them their score keys back, which
  // the masses of the dispersion curves and the coverage prefix read.
  for (int t = threadIdx.x; t < g.keep_w; t += kSortThreads)
    keys_out[base + t] = desc_key(scores[base + n - g.keep_w + t]);
}

// The counters of a 1024-thread workgroup that ranks up to kSortRun elements
// by an 8-bit digit, element (wave R + r) 64 + lane in round r of its wave.
struct RankLds {
  uint32_t start[256];  // digit-major start of each digit among the elements
  uint32_t tot[256];    // elements of each digit
  alignas(16) uint32_t wave_cnt[kSortWaves][256];  // also read and written 16 bytes at a time
};
constexpr int kRunRounds = kSortRun / kSortThreads;

__device__ __forceinline__ void rank_clear(RankLds& s, int lane, int wave) {
  if (threadIdx.x < 256) s.tot[threadIdx.x] = 0u;
#pragma unroll
  for (int j = 0; j < 4; ++j) s.wave_cnt[wave][lane * 4 + j] = 0u;
}

// Stable digit-major position of each of this thread's R <= kRunRounds
// elements (valid below cnt) among the workgroup's; the counters are clear on
// entry, and every thread is past a barrier between their clearing and this.
// Ends past a barrier, with start[] and tot[] in place.
__device__ __forceinline__ void rank_digits(RankLds& s, const uint32_t (&dg)[kRunRounds], int R,
                                            int cnt, int lane, int wave,
                                            uint32_t (&lp)[kRunRounds]) {
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r) {
    if (r < R) {
      const bool ok = (wave * R + r) * 64 + lane < cnt;
      const uint64_t peers = match_digit(dg[r], ok);
      const uint32_t below = count_below(peers);
      uint32_t pre = 0;
      if (ok) pre = s.wave_cnt[wave][dg[r]];
      lp[r] = pre + below;
      if (ok && below == 0) {
        const uint32_t c = (uint32_t)__popcll(peers);
        s.wave_cnt[wave][dg[r]] = pre + c;
        atomicAdd(&s.tot[dg[r]], c);
      }
    }
  }
  __syncthreads();
  if (wave == 0) {
    for (int j = 0; j < 4; ++j) s.start[lane * 4 + j] = s.tot[lane * 4 + j];
    wave_scan256(s.start, lane);
  } else if (threadIdx.x >= 256 && threadIdx.x < 512) {
    const int d = threadIdx.x - 256;
    uint32_t c[kSortWaves];
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) c[w] = s.wave_cnt[w][d];
    uint32_t acc = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
      s.wave_cnt[w][d] = acc;
      acc += c[w];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r)
    if (r < R && (wave * R + r) * 64 + lane < cnt)
      lp[r] += s.start[dg[r]] + s.wave_cnt[wave][dg[r]];
}

// (key, position) as one word: the order of the sort.
__device__ __forceinline__ uint64_t sort_word(uint32_t key, int pos) {
  return ((uint64_t)key << 32) | (uint32_t)pos;
}

struct OrderLds {
  RankLds rk;               // also the cells' counters, then their starts
  uint64_t word[kSortRun];  // the elements
  float sum[kSortWaves], dev[kSortWaves];
  uint32_t tot[kSortWaves];
  uint32_t crowded;
};
constexpr int kCells = kSortRun;
constexpr int kCellMax = 96;
static_assert(sizeof(((RankLds*)0)->wave_cnt) == kCells * 4, "one counter per cell");

// Where the cells of a sort lie: cell (d - low) scale, clamped, for a key d
// above the reference.
struct CellMap {
  uint32_t ref;
  float low, scale;
  // key minus the reference, clamped to 30 bits: grows with the key
  __device__ __forceinline__ float diff(uint32_t k) const {
    return k >= ref ? (float)(int)min(k - ref, 0x3fffffffu)
                    : -(float)(int)min(ref - k, 0x3fffffffu);
  }
  __device__ __forceinline__ uint32_t cell(uint32_t k) const {
    return (uint32_t)fminf(fmaxf((diff(k) - low) * scale, 0.f), (float)(kCells - 1));
  }
};

// Cells over the mean +- five mean deviations of a workgroup's keys (a few
// scores far above the others don't widen the cells).
__device__ __forceinline__ CellMap cells_around_mean(OrderLds& s, const uint32_t (&key)[kRunRounds],
                                                     uint32_t ref, int R, int cnt, int lane,
                                                     int wave) {
  CellMap cm{ref, 0.f, 0.f};
  auto valid = [&](int r) { return r < R && (wave * R + r) * 64 + lane < cnt; };
  float x = 0.f;
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r)
    if (valid(r)) x += cm.diff(key[r]);
  x = wave_sum(x);
  if (lane == 0) s.sum[wave] = x;
  __syncthreads();
  float mean = 0.f;
#pragma unroll
  for (int w = 0; w < kSortWaves; ++w) mean += s.sum[w];
  mean /= (float)cnt;
  x = 0.f;
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r)
    if (valid(r)) x += fabsf(cm.diff(key[r]) - mean);
  x = wave_sum(x);
  if (lane == 0) s.dev[wave] = x;
  __syncthreads();
  float dev = 0.f;
#pragma unroll
  for (int w = 0; w < kSortWaves; ++w) dev += s.dev[w];
  dev /= (float)cnt;
  cm.low = mean - 5.f * dev;
  cm.scale = dev > 0.f ? (float)kCells / (10.f * dev) : 0.f;
  return cm;
}

// Order cnt <= kSortRun elements in LDS by (key, position).  They come in
// registers, element (wave R + r) 64 + lane in round r of R = ceil(cnt / 1024),
// in position order; they end in s.word, past a barrier.
// The elements are dealt into kCells cells by key (those beyond the cells'
// range into the end ones), and an element's place is its cell's start plus
// the elements of the cell below it: with about one element per cell that is
// a couple of LDS reads.  Four counting passes take 4 x 8 ballots per element,
// which bind the vector unit (buckets of 64 units of 65536 keys, 1365 each: 113
// us with them, 67 us with cells; 40 us with 2048 each and two workgroups to a
// compute unit).  They are left for a cell of more than kCellMax elements:
// many equal or close keys beside far ones.  (Not unrolled: four copies spill at
// the 64 VGPRs of two workgroups to a compute unit.)
__device__ __forceinline__ void lds_order(OrderLds& s, const uint32_t (&key)[kRunRounds],
                                          const int32_t (&val)[kRunRounds], const CellMap& cm,
                                          int R, int cnt, int lane, int wave) {
  uint32_t* cell = &s.rk.wave_cnt[0][0];
  const int tid = threadIdx.x;
  auto valid = [&](int r) { return r < R && (wave * R + r) * 64 + lane < cnt; };
  reinterpret_cast<uint4*>(cell)[tid] = make_uint4(0u, 0u, 0u, 0u);
  if (tid == 0) s.crowded = 0u;
  __syncthreads();
  uint32_t cs[kRunRounds];  // cell, and the place in it above
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r) {
    if (valid(r)) {
      const uint32_t c = cm.cell(key[r]);
      cs[r] = c | atomicAdd(&cell[c], 1u) << 16;
    }
  }
  __syncthreads();
  // exclusive scan of the counters, four per thread
  {
    const uint4 x = reinterpret_cast<const uint4*>(cell)[tid];
    const uint32_t t = x.x + x.y + x.z + x.w;
    uint32_t incl = t;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    if (lane == 63) s.tot[wave] = incl;
    if (max(max(x.x, x.y), max(x.z, x.w)) > (uint32_t)kCellMax) s.crowded = 1u;
    __syncthreads();
    uint32_t e = incl - t;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) e += w < wave ? s.tot[w] : 0u;
    reinterpret_cast<uint4*>(cell)[tid] = make_uint4(e, e + x.x, e + x.x + x.y, e + x.x + x.y + x.z);
  }
  const bool crowded = s.crowded != 0u;
  __syncthreads();
  if (!crowded) {
#pragma unroll
    for (int r = 0; r < kRunRounds; ++r)
      if (valid(r)) s.word[cell[cs[r] & 0xffffu] + (cs[r] >> 16)] = sort_word(key[r], val[r]);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRunRounds; ++r) {
      if (valid(r)) {
        const uint64_t me = sort_word(key[r], val[r]);
        const uint32_t c = cs[r] & 0xffffu;
        const int i0 = (int)cell[c], i1 = c + 1 < (uint32_t)kCells ? (int)cell[c + 1] : cnt;
        uint32_t at = (uint32_t)i0;
        for (int i = i0; i < i1; ++i) at += s.word[i] < me ? 1u : 0u;
        cs[r] = at;
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRunRounds; ++r)
      if (valid(r)) s.word[cs[r]] = sort_word(key[r], val[r]);
    __syncthreads();
    return;
  }
  uint32_t k[kRunRounds];
  int32_t v[kRunRounds];
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r) {
    k[r] = key[r];
    v[r] = val[r];
  }
#pragma unroll 1
  for (int p = 0; p < 4; ++p) {
    rank_clear(s.rk, lane, wave);
    __syncthreads();
    uint32_t dg[kRunRounds], lp[kRunRounds];
#pragma unroll
    for (int r = 0; r < kRunRounds; ++r) dg[r] = (k[r] >> (8 * p)) & 255u;
    rank_digits(s.rk, dg, R, cnt, lane, wave, lp);
#pragma unroll
    for (int r = 0; r < kRunRounds; ++r)
      if (valid(r)) s.word[lp[r]] = sort_word(k[r], v[r]);
    __syncthreads();
    if (p < 3) {
#pragma unroll
      for (int r = 0; r < kRunRounds; ++r) {
        if (valid(r)) {
          const uint64_t x = s.word[(wave * R + r) * 64 + lane];
          k[r] = (uint32_t)(x >> 32);
          v[r] = (int32_t)(uint32_t)x;
        }
      }
    }
  }
}

// Sum of (s)_+ of a thread's scores over the workgroup, in thread 0.
__device__ __forceinline__ double block_sum(double x, double* red, int lane, int wave) {
  x = wave_sum(x);
  if (lane == 0) red[wave] = x;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < kSortWaves; ++w) t += red[w];
  return t;
}

// Units of at most kSortRun elements: one LDS sort each.
__global__ __launch_bounds__(kSortThreads) void sort_small_kernel(
    Geo g, SeqTab st, const float* __restrict__ scores, uint32_t* __restrict__ keys_out,
    int32_t* __restrict__ perm_out, double* __restrict__ ssum_out) {
  __shared__ OrderLds so;
  __shared__ double red[kSortWaves];
  const int h = blockIdx.x % g.H;
  const int bl = blockIdx.x / g.H;
  const int l = blockIdx.y;
  if (bl >= st.count) return;
  const int n = st.len[bl];
  const int64_t base = lht_base(g, l, h, st.start[bl]);
  const int64_t u = unit_index(g, l, st.first + bl, h);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wkeep = n - g.keep_w;
  const int R = (n + kSortThreads - 1) / kSortThreads;
  const BufRsrc srs = make_rsrc(scores + base, (uint32_t)n * 4u);
  uint32_t key[kRunRounds];
  int32_t val[kRunRounds];
  double psum = 0.0;
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r) {
    val[r] = (wave * R + r) * 64 + lane;
    key[r] = r < R ? buf_load_u32(srs, (uint32_t)val[r] * 4u) : 0u;  // past n: zero
  }
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r) {
    const float s = __uint_as_float(key[r]);
    if (s > 0.f) psum += (double)s;
    key[r] = val[r] >= wkeep ? 0u : desc_key(s);
  }
  const double tot = block_sum(psum, red, lane, wave);
  if (threadIdx.x == 0) ssum_out[u] = tot;
  const CellMap cm = cells_around_mean(so, key, desc_key(scores[base]), R, n, lane, wave);
  lds_order(so, key, val, cm, R, n, lane, wave);
  for (int i = threadIdx.x; i < n; i += kSortThreads) {
    const uint64_t x = so.word[i];
    const int32_t v = (int32_t)(uint32_t)x;
    // (a kept window's key is its score's again in the final order)
    keys_out[base + i] = v >= wkeep ? desc_key(scores[base + v]) : (uint32_t)(x >> 32);
    perm_out[base + i] = v;
  }
}

// Position of sample i of ns among n: one of every n / ns positions, chosen by
// a mix of the sample's number.  At even steps, scores with a period (pages, turns of a
// dialogue) whose multiple the step is would show the samples one phase only
// and leave the rest in a few buckets that outgrow LDS (256 units of 131072, every
// 64th score low: a selection 24980 us, 677 so; 720 with one workgroup per unit).
__device__ __forceinline__ int sort_sample(int i, int n, int ns) {
  // (below 2^31: at most 4096 samples of 262144 positions)
  const uint32_t lo = (uint32_t)i * n / ns, hi = (uint32_t)(i + 1) * n / ns;
  uint32_t x = (uint32_t)i * 0x9e3779b1u;
  x = (x ^ x >> 15) * 0x2c1b3c6du;
  x ^= x >> 13;
  return (int)(lo + __umulhi(x, hi - lo));
}

__global__ __launch_bounds__(kSortThreads) void sort_splitters_kernel(
    Geo g, SeqTab st, const float* __restrict__ scores, uint64_t* __restrict__ splitters,
    uint2* __restrict__ windows) {
  __shared__ OrderLds so;
  const int h = blockIdx.x % g.H;
  const int bl = blockIdx.x / g.H;
  const int l = blockIdx.y;
  if (bl >= st.count) return;
  const int n = st.len[bl];
  const int nb = sort_nb(n);
  if (nb <= 1) return;
  const int64_t base = lht_base(g, l, h, st.start[bl]);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wkeep = n - g.keep_w;
  const int ns = nb * kSortOver;  // <= kSortRun, < n
  const int R = (ns + kSortThreads - 1) / kSortThreads;
  uint32_t key[kRunRounds];
  int32_t val[kRunRounds];
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r) {
    const int i = min((wave * R + r) * 64 + lane, ns - 1);
    val[r] = sort_sample(i, n, ns);  // ascending: equal keys stay in position order
    key[r] = r < R ? __float_as_uint(scores[base + val[r]]) : 0u;
  }
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r)
    key[r] = val[r] >= wkeep ? 0u : desc_key(__uint_as_float(key[r]));
  const CellMap cm = cells_around_mean(so, key, desc_key(scores[base]), R, ns, lane, wave);
  lds_order(so, key, val, cm, R, ns, lane, wave);
  if (threadIdx.x < nb) {
    const int64_t b0 = part_base(g, st, l, bl, h, [&](int i) { return sort_nb(st.len[i]); });
    const int i = threadIdx.x * kSortOver;
    if (threadIdx.x > 0) splitters[b0 + threadIdx.x - 1] = so.word[i];
    // the second and the second to last sample of the bucket: its cells reach
    // as far again on either side (one stray sample doesn't widen them)
    windows[b0 + threadIdx.x] = make_uint2((uint32_t)(so.word[i + 1] >> 32),
                                                   (uint32_t)(so.word[i + kSortOver - 2] >> 32));
  }
}

// Buckets of a tile's elements (8 bits each, to ids) and their counts, and the
// tile's sum of (s)_+.
__global__ __launch_bounds__(kSortThreads) void sort_count_kernel(
    Geo g, SeqTab st, int32_t nb_max, const float* __restrict__ scores,
    const uint64_t* __restrict__ splitters, uint8_t* __restrict__ ids,
    uint32_t* __restrict__ counts, double* __restrict__ tile_sum) {
  __shared__ uint64_t sp[256];
  __shared__ uint32_t cnt_s[256];
  __shared__ double red[kSortWaves];
  int h, tile;
  const int bl = locate_part(
      g, st, blockIdx.x, [&](int i) { return sort_tiles(st.len[i]); }, h, tile);
  const int l = blockIdx.y;
  if (bl >= st.count) return;
  const int n = st.len[bl];
  const int e0 = tile * kSortRun;
  const int nb = sort_nb(n);
  const int64_t base = lht_base(g, l, h, st.start[bl]);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wkeep = n - g.keep_w;
  const BufRsrc srs = make_rsrc(scores + base, (uint32_t)n * 4u);
  uint32_t raw[kRunRounds];
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r)
    raw[r] = buf_load_u32(srs, (uint32_t)(e0 + r * kSortThreads + tid) * 4u);
  // (while the scores are on their way)
  const int64_t b0 = part_base(g, st, l, bl, h, [&](int i) { return sort_nb(st.len[i]); });
  const int64_t t0 = part_base_of(g, l, blockIdx.x, tile, sort_tiles(n));
  if (tid < nb) {
    sp[tid] = tid < nb - 1 ? splitters[b0 + tid] : ~0ull;
    cnt_s[tid] = 0u;
  }
  __syncthreads();
  int step0 = 1;
  while (step0 * 2 < nb) step0 *= 2;  // largest power of two below nb
  double psum = 0.0;
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r) {
    const int e = e0 + r * kSortThreads + tid;
    const float s = __uint_as_float(raw[r]);
    if (s > 0.f) psum += (double)s;
    const uint64_t w = sort_word(e >= wkeep ? 0u : desc_key(s), e);
    int b = 0;  // splitters at or below w
    if (nb > 1)
      for (int d = step0; d > 0; d >>= 1)
        if (b + d <= nb - 1 && sp[b + d - 1] <= w) b += d;
    if (e < n) {
      ids[base + e] = (uint8_t)b;
      atomicAdd(&cnt_s[b], 1u);
    }
  }
  const double t = block_sum(psum, red, lane, wave);  // past a barrier: the counts are whole
  if (tid == 0) tile_sum[t0 + tile] = t;
  if (tid < nb) counts[(t0 + tile) * nb_max + tid] = cnt_s[tid];
}

// Elements of a tile to their buckets, in position order: ranks by bucket as
// in a radix pass, staged bucket-major so that runs are written together.
__global__ __launch_bounds__(kSortThreads) void sort_scatter_kernel(
    Geo g, SeqTab st, int32_t nb_max, const float* __restrict__ scores,
    const uint8_t* __restrict__ ids, const uint32_t* __restrict__ counts,
    const double* __restrict__ tile_sum, uint32_t* __restrict__ keys, int32_t* __restrict__ vals,
    uint32_t* __restrict__ bucket_start, double* __restrict__ ssum_out) {
  __shared__ RankLds rk;
  __shared__ uint32_t skey[kSortRun];
  __shared__ uint16_t soff[kSortRun];   // position within the tile
  __shared__ uint8_t sid[kSortRun];
  __shared__ uint32_t bstart[256], before[256];
  int h, tile;
  const int bl = locate_part(
      g, st, blockIdx.x, [&](int i) { return sort_tiles(st.len[i]); }, h, tile);
  const int l = blockIdx.y;
  if (bl >= st.count) return;
  const int n = st.len[bl];
  const int e0 = tile * kSortRun;
  const int nb = sort_nb(n);
  const int ntile = sort_tiles(n);
  const int cnt = min(kSortRun, n - e0);
  const int64_t base = lht_base(g, l, h, st.start[bl]);
  const int64_t u = unit_index(g, l, st.first + bl, h);
  const int64_t t0 = part_base_of(g, l, blockIdx.x, tile, ntile);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wkeep = n - g.keep_w;
  uint32_t raw[kRunRounds], dg[kRunRounds], lp[kRunRounds];
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r) {
    const int e = min(e0 + (wave * kRunRounds + r) * 64 + lane, n - 1);
    raw[r] = __float_as_uint(scores[base + e]);
    dg[r] = ids[base + e];
  }
  // bucket totals over the tiles, and the counts of the tiles before this
  // one: thread d of the first 256 takes a bucket
  if (tid < 256) {
    uint32_t all = 0u, bef = 0u;
    if (tid < nb) {
      const uint32_t* c = counts + t0 * nb_max + tid;
#pragma unroll 8
      for (int t = 0; t < ntile; ++t) {
        const uint32_t x = c[(int64_t)t * nb_max];
        all += x;
        bef += t < tile ? x : 0u;
      }
    }
    bstart[tid] = all;
    before[tid] = bef;
  }
  rank_clear(rk, lane, wave);
  __syncthreads();
  if (wave == 15) wave_scan256(bstart, lane);  // read after the ranking's barriers
  rank_digits(rk, dg, kRunRounds, cnt, lane, wave, lp);
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r) {
    const int x = (wave * kRunRounds + r) * 64 + lane;
    if (x < cnt) {
      skey[lp[r]] = e0 + x >= wkeep ? 0u : desc_key(__uint_as_float(raw[r]));
      soff[lp[r]] = (uint16_t)x;
      sid[lp[r]] = (uint8_t)dg[r];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRunRounds; ++r) {
    const int i = tid + r * kSortThreads;
    if (i < cnt) {
      const uint32_t d = sid[i];
      const uint32_t dst = bstart[d] + before[d] + (uint32_t)i - rk.start[d];
      keys[base + dst] = skey[i];
      vals[base + dst] = e0 + (int)soff[i];
    }
  }
  if (tile == 0) {
    const int64_t b0 = part_base(g, st, l, bl, h, [&](int i) { return sort_nb(st.len[i]); });
    if (tid < nb) bucket_start[b0 + tid] = bstart[tid];
    if (wave == 1) {
      double x = 0.0;
      for (int t = lane; t < ntile; t += 64) x += tile_sum[t0 + t];
      x = wave_sum(x);
      if (lane == 0) ssum_out[u] = x;
    }
  }
}

// (eight waves per SIMD: two workgroups to a compute unit)
__global__ __launch_bounds__(kSortThreads)
__attribute__((amdgpu_waves_per_eu(8, 8))) void sort_buckets_kernel(
    Geo g, SeqTab st, const float* __restrict__ scores,
    uint32_t* __restrict__ keys_in, int32_t* __restrict__ vals_in,
    const uint32_t* __restrict__ bucket_start, const uint2* __restrict__ windows,
    uint32_t* __restrict__ keys_out, int32_t* __restrict__ perm_out) {
  __shared__ OrderLds so;
  RankLds& rk = so.rk;
  __shared__ uint32_t place[256];  // next place of each digit (sorts through memory)
  int h, bk;
  const int bl = locate_part(
      g, st, blockIdx.x, [&](int i) { return sort_nb(st.len[i]); }, h, bk);
  const int l = blockIdx.y;
  if (bl >= st.count) return;
  const int n = st.len[bl];
  const int nb = sort_nb(n);
  const int64_t base = lht_base(g, l, h, st.start[bl]);
  const int64_t b0 = part_base_of(g, l, blockIdx.x, bk, nb);
  const int lo = (int)bucket_start[b0 + bk];
  const int m = (bk + 1 < nb ? (int)bucket_start[b0 + bk + 1] : n) - lo;
  if (m <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wkeep = n - g.keep_w;
  uint32_t* ka = keys_in + base + lo;
  int32_t* va = vals_in + base + lo;
  uint32_t* kb = keys_out + base + lo;
  int32_t* vb = perm_out + base + lo;
  // final order of element i: (a kept window's key is its score's again)
  auto emit = [&](int i, uint32_t k, int32_t v) {
    kb[i] = v >= wkeep ? desc_key(scores[base + v]) : k;
    vb[i] = v;
  };
  uint32_t key[kRunRounds];
  int32_t val[kRunRounds];
  if (m <= kSortRun) {
    const int R = (m + kSortThreads - 1) / kSortThreads;
#pragma unroll
    for (int r = 0; r < kRunRounds; ++r) {
      const int i = min((wave * R + r) * 64 + lane, m - 1);
      key[r] = ka[i];
      val[r] = va[i];
    }
    CellMap cm;
    if (nb > 1) {
      const uint2 w = windows[b0 + bk];
      const float span = (float)(w.y - w.x);
      cm = CellMap{w.x, -span, (float)kCells / (3.f * span + 1.f)};
    } else {
      cm = cells_around_mean(so, key, ka[0], R, m, lane, wave);
    }
    lds_order(so, key, val, cm, R, m, lane, wave);
    for (int i = tid; i < m; i += kSortThreads) {
      const uint64_t x = so.word[i];
      emit(i, (uint32_t)(x >> 32), (int32_t)(uint32_t)x);
    }
    return;
  }
  // Through memory: four counting passes over tiles, between the two buffers
  // (only this workgroup touches this part of them).
  for (int p = 0; p < 4; ++p) {
    const uint32_t* kin = p & 1 ? kb : ka;
    const int32_t* vin = p & 1 ? vb : va;
    uint32_t* kout = p & 1 ? ka : kb;
    int32_t* vout = p & 1 ? va : vb;
    const int sh = 8 * p;
    if (tid < 256) place[tid] = 0u;
    __syncthreads();
    for (int i = tid; i < m; i += kSortThreads) atomicAdd(&place[(kin[i] >> sh) & 255u], 1u);
    __syncthreads();
    if (wave == 0) wave_scan256(place, lane);
    for (int t0 = 0; t0 < m; t0 += kSortRun) {
      const int cnt = min(kSortRun, m - t0);
      uint32_t dg[kRunRounds], lp[kRunRounds];
#pragma unroll
      for (int r = 0; r < kRunRounds; ++r) {
        const int i = min(t0 + (wave * kRunRounds + r) * 64 + lane, m - 1);
        key[r] = kin[i];
        val[r] = vin[i];
        dg[r] = (key[r] >> sh) & 255u;
      }
      rank_clear(rk, lane, wave);
      __syncthreads();
      rank_digits(rk, dg, kRunRounds, cnt, lane, wave, lp);
#pragma unroll
      for (int r = 0; r < kRunRounds; ++r) {
        if ((wave * kRunRounds + r) * 64 + lane < cnt) {
          const uint32_t dst = place[dg[r]] + lp[r] - rk.start[dg[r]];
          kout[dst] = key[r];
          vout[dst] = val[r];
        }
      }
      __syncthreads();
      if (tid < 256) place[tid] += rk.tot[tid];
      __syncthreads();
    }
    __threadfence_block();
    __syncthreads();  // the pass's output is the next pass's input
  }
  for (int i = tid; i < m; i += kSortThreads) emit(i, ka[i], va[i]);
}

certkv_status run_sort(const SortArgs& a, const SeqTab& st, hipStream_t s) {
  const Geo& g = a.g;
  const dim3 units(g.H * st.count, g.L);
  if (a.nb_max == 0) {
    CERTKV_LAUNCH("sort_segments", seg_sort_kernel, units, dim3(kSortThreads), 0, s, g, st,
                  a.scores, a.keysA, a.valsA, a.keysB, a.valsB, a.keys_out, a.perm_out, a.ssum);
    return CERTKV_OK;
  }
  if (a.nb_max == 1) {
    CERTKV_LAUNCH("sort_small", sort_small_kernel, units, dim3(kSortThreads), 0, s, g, st, a.scores,
                  a.keys_out, a.perm_out, a.ssum);
    return CERTKV_OK;
  }
  uint8_t* ids = reinterpret_cast<uint8_t*>(a.valsA);  // dead before the buckets are written
  const dim3 tiles(count_parts(g, st, [&](int i) { return sort_tiles(st.len[i]); }), g.L);
  CERTKV_LAUNCH("sort_splitters", sort_splitters_kernel, units, dim3(kSortThreads), 0, s, g, st,
                a.scores, a.splitters, a.windows);
  CERTKV_LAUNCH("sort_count", sort_count_kernel, tiles, dim3(kSortThreads), 0, s, g, st,
                a.nb_max, a.scores, (const uint64_t*)a.splitters, ids, a.counts,
                a.tile_sum);
  CERTKV_LAUNCH("sort_scatter", sort_scatter_kernel, tiles, dim3(kSortThreads), 0, s, g, st,
                a.nb_max, a.scores, (const uint8_t*)ids, (const uint32_t*)a.counts,
                (const double*)a.tile_sum, a.keysB, a.valsB, a.bucket_start, a.ssum);
  CERTKV_LAUNCH("sort_buckets", sort_buckets_kernel,
                dim3(count_parts(g, st, [&](int i) { return sort_nb(st.len[i]); }), g.L),
                dim3(kSortThreads), 0, s, g, st, a.scores, a.keysB, a.valsB,
                (const uint32_t*)a.bucket_start, (const uint2*)a.windows, a.keys_out, a.perm_out);
  return CERTKV_OK;
}

}  // namespace certkv
