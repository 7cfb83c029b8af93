// Kept-key selection: threshold on the score order plus ballot compaction.
//
// The top-b keys of a unit (score descending, ties by position) are exactly
// the keys whose (radix key, position) pair is lexicographically <= the pair
// at rank b-1 of the sort.  A workgroup streams its part of the unit's scores in
// position order (tiles of 8192 positions), tests each key against that
// threshold, and compacts the kept positions with wave ballots and a prefix over
// the 16 waves, so kept indices come out ascending without a scatter.  The same
// pass sums (s)_+ over the evicted keys and over all keys in fp64 (the tail mass
// and its normalizer).
#include <type_traits>

#include "stages.h"

namespace certkv {

// budgets clamped to [0, n_b] (caller-supplied budgets in selection mode)
__global__ void clamp_budgets_kernel(Geo g, SeqTab st, int32_t* __restrict__ budgets) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int per_layer = st.count * g.H;
  if (i >= per_layer * g.L) return;
  const int l = i / per_layer, r = i % per_layer;
  const int bl = r / g.H, h = r % g.H;
  const int64_t u = unit_index(g, l, st.first + bl, h);
  int32_t b = budgets[u];
  b = b < 0 ? 0 : (b > st.len[bl] ? st.len[bl] : b);
  budgets[u] = b;
}

// Exclusive prefix over all units of the budgets -> kept_offsets[U+1];
// packed_offsets[u] = kept_offsets[u] + slot * u (slot = 1: one slot row per
// unit; 0 without the slot).
__global__ __launch_bounds__(1024) void offsets_kernel(int64_t U, int32_t slot,
                                                       const int32_t* __restrict__ budgets,
                                                       int64_t* __restrict__ kept_offsets,
                                                       int64_t* __restrict__ packed_offsets) {
  __shared__ int64_t wsum[16];
  __shared__ int64_t carry;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int64_t base = 0; base < U; base += 1024) {
    const int64_t i = base + threadIdx.x;
    int64_t v = i < U ? (int64_t)budgets[i] : 0;
    int64_t incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      int64_t y = __shfl_up(incl, off, 64);
      if (lane >= off) incl += y;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int64_t before = carry;
    for (int w = 0; w < wave; ++w) before += wsum[w];
    if (i < U) {
      kept_offsets[i] = before + incl - v;
      if (packed_offsets) packed_offsets[i] = before + incl - v + slot * i;
    }
    __syncthreads();
    if (threadIdx.x == 1023) carry = before + incl;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    kept_offsets[U] = carry;
    if (packed_offsets) packed_offsets[U] = carry + slot * U;
  }
}

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelRounds = 8;                     // rounds of 1024 consecutive positions
constexpr int kSelTile = kSelThreads * kSelRounds; // 8192 positions per iteration
// Parts of a unit of n positions.
__host__ __device__ inline int sel_parts(int n, int part_tiles) {
  const int tiles = (int)(((int64_t)n + kSelTile - 1) / kSelTile);
  return (tiles + part_tiles - 1) / part_tiles;
}
constexpr int kSelScanPer = kSelRounds * kSelWaves / 64;  // counts per lane of the scan

// One workgroup per part of a unit: part_tiles tiles, or the whole unit.  Tile
// after tile with two barriers each, a long unit is a serial chain (4 us a
// tile); a part instead counts the kept keys before it by itself, from scores
// that the L2 holds, which needs no barrier and no exchange between workgroups.
// The last part meets every score that way, in the order and on the threads of
// a workgroup that walks the whole unit, and forms the sums.  Whole units and parts: 8 of 32768 positions
// 19 and 15 us, 64 of 8192 to 65536 34 and 26, 24 of 9999 to 30001 without sums
// 18 and 14.
// Whole units, sums and the mask are compile-time forms: the tests for them in
// the tile's rounds keep these from being scheduled together (256 units of 131072
// positions 72 us with the tests and 64 without; with the sums, in a pass, 81 and 71).
template <bool WHOLE, bool SUMS, bool MASK>
__global__ __launch_bounds__(kSelThreads) void select_kernel(
    Geo g, SeqTab st, int32_t part_tiles, const float* __restrict__ scores,
    const uint32_t* __restrict__ sorted_keys, const int32_t* __restrict__ perm,
    const int32_t* __restrict__ budgets, bool own_offsets, int64_t* __restrict__ kept_offsets,
    int64_t* __restrict__ packed_offsets, int32_t* __restrict__ kept_idx, int64_t capacity,
    double* __restrict__ evicted_sum, double* __restrict__ total_sum, uint64_t* __restrict__ bm,
    int32_t bm_stride, uint8_t* __restrict__ mask) {
  // kept counts of each (round, wave) of a tile, then their exclusive prefix
  // in position order (round-major); the tile's total at the end
  __shared__ uint32_t kcnt[kSelRounds * kSelWaves + 1];
  __shared__ double dsum[2][kSelWaves];
  __shared__ int64_t osum[kSelWaves];
  int h = blockIdx.x % g.H, part = 0, bl = blockIdx.x / g.H;
  if constexpr (!WHOLE)
    bl = locate_part(g, st, blockIdx.x, [&](int x) { return sel_parts(st.len[x], part_tiles); }, h,
                     part);
  const int l = blockIdx.y;
  if (bl >= st.count) return;
  const int b = st.first + bl;
  const int n = st.len[bl];
  const int64_t base = lht_base(g, l, h, st.start[bl]);
  const int64_t u = unit_index(g, l, b, h);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int bb = budgets[u];
  const int wkeep = n - g.keep_w;  // first kept-window position (n: none)
  uint32_t kthr = 0u;
  int32_t ithr = -1;  // keep nothing when bb == 0
  if (bb > 0 && bb <= n) {
    kthr = sorted_keys[base + bb - 1];
    ithr = perm[base + bb - 1];
  }
  // Round r of a tile: positions j0 + 1024 r + thread, so every load covers
  // 256 consecutive bytes per wave.  Loads through a range-checked buffer:
  // positions past the end read as zero, so no branch sits around them and
  // the next tile's loads stay in flight while this one is tested; they are
  // masked where used.
  const BufRsrc srs = make_rsrc(scores + base, (uint32_t)n * 4u);
  auto load = [&](int j0, float (&sv)[kSelRounds]) {
#pragma unroll
    for (int r = 0; r < kSelRounds; ++r)
      sv[r] = __uint_as_float(
          buf_load_u32(srs, (uint32_t)(j0 + r * kSelThreads + (int)threadIdx.x) * 4u));
  };
  const int start = WHOLE ? 0 : (int)min((int64_t)part * part_tiles * kSelTile, (int64_t)n);
  const int end = WHOLE ? n : (int)min((int64_t)(part + 1) * part_tiles * kSelTile, (int64_t)n);
  const bool sums = SUMS && (WHOLE || end == n);  // the unit's last part
  float cur[kSelRounds], nxt[kSelRounds];
  load(start, cur);
  int64_t off = 0;
  if (own_offsets) {
    // the budgets before this unit's, summed by every workgroup (kSelOwnOffsets
    // at most: one load a thread); a unit's first part writes its offsets
    const int64_t v = wave_sum((int64_t)((int64_t)threadIdx.x < u ? budgets[threadIdx.x] : 0));
    if (lane == 0) osum[wave] = v;
    __syncthreads();
    for (int w = 0; w < kSelWaves; ++w) off += osum[w];
    if (part == 0 && threadIdx.x == 0) {
      kept_offsets[u] = off;
      if (packed_offsets) packed_offsets[u] = off + g.slot * u;
      const int64_t U = (int64_t)g.L * g.B * g.H;
      if (u == U - 1) {
        kept_offsets[U] = off + bb;
        if (packed_offsets) packed_offsets[U] = off + bb + g.slot * U;
      }
    }
  } else {
    off = kept_offsets[u];
  }
  int64_t run = 0;
  double se = 0.0, sa = 0.0;
  // kept window keys hold ranks 0..w-1 in position order; the others are kept up
  // to the threshold pair at rank bb-1
  auto keeps = [&](int j, float x) -> bool {
    const uint32_t key = desc_key(x);
    return j < n && (j >= wkeep ? (j - wkeep < bb)
                                : (bb > g.keep_w && (key < kthr || (key == kthr && j <= ithr))));
  };
  if (!WHOLE && start > 0) {
    uint32_t before = 0;
    float x[kSelRounds], y[kSelRounds];
    load(0, x);
    for (int j0 = 0; j0 < start; j0 += kSelTile) {
      load(j0 + kSelTile, y);  // (of the part itself, unused, after the last tile)
#pragma unroll
      for (int r = 0; r < kSelRounds; ++r) {
        const bool keep = keeps(j0 + r * kSelThreads + (int)threadIdx.x, x[r]);
        before += keep ? 1u : 0u;
        if (sums) {
          const double sp = x[r] > 0.f ? (double)x[r] : 0.0;
          sa += sp;
          se += keep ? 0.0 : sp;
        }
      }
#pragma unroll
      for (int r = 0; r < kSelRounds; ++r) x[r] = y[r];
    }
    const uint32_t c = wave_sum(before);
    if (lane == 0) kcnt[wave] = c;
    __syncthreads();
    for (int w = 0; w < kSelWaves; ++w) run += kcnt[w];
    __syncthreads();
  }
  for (int j0 = start; j0 < end; j0 += kSelTile) {
    load(j0 + kSelTile, nxt);
    uint32_t kmask = 0;
    uint64_t bal[kSelRounds];  // wave-uniform: scalar registers
#pragma unroll
    for (int r = 0; r < kSelRounds; ++r) {
      const int j = j0 + r * kSelThreads + (int)threadIdx.x;
      const bool valid = j < n;
      const bool keep = keeps(j, cur[r]);
      if (sums) {
        const double sp = (valid && cur[r] > 0.f) ? (double)cur[r] : 0.0;
        sa += sp;
        se += keep ? 0.0 : sp;
      }
      bal[r] = __ballot(keep);
      if (MASK && valid) mask[base + j] = keep ? 1 : 0;  // 64 consecutive bytes per wave
      kmask |= (uint32_t)keep << r;
      if (lane == 0) {
        kcnt[r * kSelWaves + wave] = (uint32_t)__popcll(bal[r]);
        // kept bitmap: the ballot is the word of the wave's 64 positions
        const int widx = ((j0 + r * kSelThreads) >> 6) + wave;
        if (bm && widx < bm_stride) bm[u * bm_stride + widx] = bal[r];
      }
    }
    __syncthreads();
    // exclusive prefix of the counts in position order (one wave)
    if (wave == 0) {
      uint32_t c[kSelScanPer], t = 0;
#pragma unroll
      for (int i = 0; i < kSelScanPer; ++i) {
        c[i] = kcnt[kSelScanPer * lane + i];
        t += c[i];
      }
      uint32_t incl = t;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
      }
      uint32_t ex = incl - t;
#pragma unroll
      for (int i = 0; i < kSelScanPer; ++i) {
        kcnt[kSelScanPer * lane + i] = ex;
        ex += c[i];
      }
      if (lane == 63) kcnt[kSelRounds * kSelWaves] = incl;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSelRounds; ++r) {
      if ((kmask >> r) & 1u) {
        const uint32_t below = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(bal[r] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal[r], 0u));
        const int64_t dst = off + run + kcnt[r * kSelWaves + wave] + below;
        if (dst < capacity) kept_idx[dst] = j0 + r * kSelThreads + (int)threadIdx.x;
      }
    }
    run += kcnt[kSelRounds * kSelWaves];
#pragma unroll
    for (int r = 0; r < kSelRounds; ++r) cur[r] = nxt[r];
  }
  if (!sums) return;
  se = wave_sum(se);
  sa = wave_sum(sa);
  if (lane == 0) {
    dsum[0][wave] = se;
    dsum[1][wave] = sa;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double e = 0.0, t = 0.0;
    for (int w = 0; w < kSelWaves; ++w) {
      e += dsum[0][w];
      t += dsum[1][w];
    }
    evicted_sum[u] = e;
    total_sum[u] = t;
  }
}

// Coverage budget k_eta: the normalizer sum (s)_+ in position order, then the
// rank-order prefix of a = (s)_+ / sum until it reaches retain, both summed
// one term at a time in fp64.  One 16-wave workgroup per unit.
//
// The serial sums are a chain of up to 2 n dependent additions, so the
// workgroup first finds the crossing from sums taken in another order: the
// total over all threads, then the rank range holding the crossing narrowed
// 16-fold per step (each wave sums one part of it) down to one wave's 64
// ranks.  With unit roundoff u = 2^-53, a prefix of at most n non-negative
// terms adding up to at most 1 is within n u of its exact value when summed
// serially, the total carries another n u into every term, the quotients u
// each, and this kernel's own sums stay within n u likewise: a prefix
// differs from the serial one by less than 4 n u.  If the prefixes on both
// sides of the crossing clear retain by twice that, the serial sums cross at
// the same rank.  Otherwise (prefixes tied with retain: flat or quantized
// scores, retain = 1, a non-finite total) the serial sums decide.
// Three sequences of 16384, 9999 and 30001 keys, two layers, 8 heads: 3740 us
// with the serial sums alone, 13 us; flat scores, which fall back: 165 us.
constexpr int kCovThreads = 1024;
constexpr int kCovWaves = kCovThreads / 64;

__global__ __launch_bounds__(kCovThreads) void coverage_kernel(
    Geo g, SeqTab st, const float* __restrict__ scores, const uint32_t* __restrict__ sorted_keys,
    double retain, int32_t* __restrict__ budgets) {
  __shared__ double wsum[kCovWaves];
  __shared__ double buf[2][kCovThreads];
  __shared__ int32_t decided, hit_at[2];
  const int h = blockIdx.x % g.H;
  const int bl = blockIdx.x / g.H;
  const int l = blockIdx.y;
  if (bl >= st.count) return;
  const int b = st.first + bl;
  const int n = st.len[bl];
  const int64_t base = lht_base(g, l, h, st.start[bl]);
  const int64_t u = unit_index(g, l, b, h);
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const BufRsrc srs = make_rsrc(scores + base, (uint32_t)n * 4u);
  const BufRsrc krs = make_rsrc(sorted_keys + base, (uint32_t)n * 4u);
  auto pos_part = [](float s) { return s > 0.f ? (double)s : 0.0; };
  // (s)_+ at rank r, zero from rank hi on (reads past n are range-checked)
  auto at_rank = [&](int r, int hi) {
    const double x = pos_part(desc_key_value(buf_load_u32(krs, (uint32_t)r * 4u)));
    return r < hi ? x : 0.0;
  };

  // total, in any order
  double part = 0.0;
#pragma unroll 8
  for (int j = tid; j < n; j += kCovThreads)
    part += pos_part(__uint_as_float(buf_load_u32(srs, (uint32_t)j * 4u)));
  part = wave_sum(part);
  if (lane == 0) wsum[wave] = part;
  __syncthreads();
  double tot = 0.0;
  for (int w = 0; w < kCovWaves; ++w) tot += wsum[w];
  __syncthreads();

  // ranks [lo, hi) hold the crossing if there is one; below: the sum before lo
  const double goal = retain * tot;
  int lo = 0, hi = n;
  double below = 0.0;
  while (hi - lo > 64) {
    const int per = ((hi - lo + kCovWaves - 1) / kCovWaves + 63) & ~63;
    const int w0 = lo + wave * per, w1 = min(hi, w0 + per);
    double x = 0.0;
#pragma unroll 8
    for (int r = w0 + lane; r < w1; r += 64) x += at_rank(r, w1);
    x = wave_sum(x);
    if (lane == 0) wsum[wave] = x;
    __syncthreads();
    int pick = kCovWaves - 1;  // no crossing: the last part, and on to rank n
    double before = below;
    for (int w = 0; w < kCovWaves; ++w) {
      if (below + wsum[w] >= goal) {
        pick = w;
        break;
      }
      below += wsum[w];
      if (w + 1 < kCovWaves) before = below;
    }
    below = before;
    const int nlo = min(hi, lo + pick * per);
    hi = min(hi, nlo + per);
    lo = nlo;
    __syncthreads();
  }
  if (wave == 0) {
    double incl = at_rank(lo + lane, hi);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const double y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    incl += below;
    double prev = __shfl_up(incl, 1, 64);
    if (lane == 0) prev = below;
    const double eps = 8.0 * (double)n * 1.1102230246251565e-16 * tot;
    // at most one lane: prefixes do not decrease.  A NaN decides nothing.
    const bool here = lane < hi - lo && incl >= goal + eps && prev < goal - eps && tot > 0.0 &&
                      tot < INFINITY;
    const uint64_t m = __ballot(here);
    if (lane == 0) decided = m ? lo + (int)__builtin_ctzll(m) + 1 : 0;
  }
  __syncthreads();
  int k = decided;
  if (k == 0) {
    // Serial sums: every thread loads one term of the next 1024 into LDS while
    // each thread adds up the current ones (the same additions everywhere: the
    // operands are LDS broadcasts and the loop ends together).
    double x[1];
    tot = 0.0;
    const int nt = (n + kCovThreads - 1) / kCovThreads;
    x[0] = pos_part(__uint_as_float(buf_load_u32(srs, (uint32_t)tid * 4u)));
    for (int t = 0; t < nt; ++t) {
      buf[t & 1][tid] = x[0];
      __syncthreads();
      x[0] = pos_part(__uint_as_float(buf_load_u32(srs, (uint32_t)((t + 1) * kCovThreads + tid) * 4u)));
      const int cnt = min(kCovThreads, n - t * kCovThreads);
      const double* q = buf[t & 1];
      if (wave == 0) {
#pragma unroll 16
        for (int i = 0; i < cnt; ++i) tot += q[i];
      }
    }
    __syncthreads();
    if (tid == 0) wsum[0] = tot;
    __syncthreads();
    tot = wsum[0];
    const double inv_n = 1.0 / (double)n;
    auto term = [&](int r) {
      const float s = desc_key_value(buf_load_u32(krs, (uint32_t)r * 4u));
      const double a = tot > 0.0 ? (s > 0.f ? (double)s / tot : 0.0) : inv_n;
      return r < n ? a : 0.0;
    };
    double p = 0.0;
    k = n;
    if (tid < 2) hit_at[tid] = 0;
    x[0] = term(tid);
    // (tile t's hit goes to slot t % 2, which is not written again before
    // every thread has passed the next barrier: all of them leave together)
    int found = 0;
    for (int t = 0; t < nt; ++t) {
      buf[t & 1][tid] = x[0];
      __syncthreads();
      found = hit_at[(t & 1) ^ 1];
      if (found) break;
      x[0] = term((t + 1) * kCovThreads + tid);
      const int cnt = min(kCovThreads, n - t * kCovThreads);
      const double* q = buf[t & 1];
      if (wave == 0) {
        // blocks of 16 additions: the prefix is monotone, so a block whose
        // end stays below retain holds no crossing
        int i = 0;
        bool hit = false;
        for (; i + 16 <= cnt; i += 16) {
          double e = p;
#pragma unroll
          for (int j = 0; j < 16; ++j) e += q[i + j];
          if (!(e < retain)) {
            hit = true;
            break;
          }
          p = e;
        }
        if (hit || i < cnt) {
          const int end = hit ? i + 16 : cnt;
          hit = false;
          for (; i < end; ++i) {
            p += q[i];
            if (p >= retain) {
              hit = true;
              break;
            }
          }
          // (a block may stop without a crossing only if a term is NaN)
          while (!hit && i < cnt) {
            p += q[i++];
            if (p >= retain) {
              hit = true;
              --i;
            }
          }
        }
        if (hit && lane == 0) hit_at[t & 1] = t * kCovThreads + i + 1;
      }
    }
    __syncthreads();
    if (!found) found = hit_at[(nt - 1) & 1];  // the last tile's
    if (found) k = found;
  }
  // a kept window leads the order and is never cut
  if (g.keep_w) k = max(k, min(g.keep_w, n));
  if (tid == 0) budgets[u] = k;
}


certkv_status run_coverage(const Geo& g, const SeqTab& st, const float* scores,
                           const uint32_t* sorted_keys, double retain, int32_t* budgets,
                           hipStream_t s) {
  CERTKV_LAUNCH("coverage_budget", coverage_kernel, dim3(g.H * st.count, g.L), dim3(kCovThreads), 0, s, g, st,
                scores, sorted_keys, retain, budgets);
  return CERTKV_OK;
}

certkv_status run_clamp(const Geo& g, const SeqTab& st, int32_t* budgets, hipStream_t s) {
  const int total = st.count * g.H * g.L;
  CERTKV_LAUNCH("clamp_budgets", clamp_budgets_kernel, dim3((total + 255) / 256), dim3(256), 0, s, g,
                st, budgets);
  return CERTKV_OK;
}

certkv_status run_offsets(int64_t U, int32_t slot, const int32_t* budgets, int64_t* kept_offsets,
                          int64_t* packed_offsets, hipStream_t s) {
  CERTKV_LAUNCH("kept_offsets", offsets_kernel, dim3(1), dim3(1024), 0, s, U, slot, budgets,
                kept_offsets, packed_offsets);
  return CERTKV_OK;
}

__global__ void packed_from_kept_kernel(int64_t U, int32_t slot,
                                        const int64_t* __restrict__ kept_offsets,
                                        int64_t* __restrict__ packed_offsets) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i <= U) packed_offsets[i] = kept_offsets[i] + slot * i;
}

certkv_status run_packed_from_kept(int64_t U, int32_t slot, const int64_t* kept_offsets,
                                   int64_t* packed_offsets, hipStream_t s) {
  CERTKV_LAUNCH("packed_offsets", packed_from_kept_kernel, dim3((unsigned)((U + 256) / 256)),
                dim3(256), 0, s, U, slot, kept_offsets, packed_offsets);
  return CERTKV_OK;
}

// True-uniform allocation (one-factor ablation): every head of a (layer,
// sequence) gets B_real / H, which the budget algebra makes whole.
__global__ void uniform_budgets_kernel(Geo g, SeqTab st, int32_t* __restrict__ budgets) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int total = st.count * g.H * g.L;
  if (i >= total) return;
  const int h = i % g.H;
  const int bi = (i / g.H) % st.count;
  const int l = i / (g.H * st.count);
  budgets[unit_index(g, l, st.first + bi, h)] = (int32_t)(st.b_real[bi] / g.H);
}

certkv_status run_uniform_budgets(const Geo& g, const SeqTab& st, int32_t* budgets, hipStream_t s) {
  const int total = st.count * g.H * g.L;
  CERTKV_LAUNCH("uniform_budgets", uniform_budgets_kernel, dim3((total + 255) / 256), dim3(256), 0,
                s, g, st, budgets);
  return CERTKV_OK;
}

certkv_status run_select(const SelectArgs& a, const SeqTab& st, hipStream_t s) {
  // The smallest parts that start together (two workgroups to a compute unit);
  // with a unit per compute unit none is split.
  int part_tiles = 1 << 18;  // n < 2^31
  if ((int64_t)a.g.L * a.g.H * st.count < 256) {
    part_tiles = 1;
    auto wgs = [&](int t) {
      return (int64_t)a.g.L * count_parts(a.g, st, [&](int bl) { return sel_parts(st.len[bl], t); });
    };
    while (wgs(part_tiles) > 512) part_tiles *= 2;
  }
  const dim3 grid(count_parts(a.g, st, [&](int bl) { return sel_parts(st.len[bl], part_tiles); }),
                  a.g.L);
  const auto launch = [&](auto kernel) -> certkv_status {
    CERTKV_LAUNCH("select", kernel, grid, dim3(kSelThreads), 0, s, a.g, st, part_tiles, a.scores,
                  a.sorted_keys, a.perm, (const int32_t*)a.budgets, a.own_offsets, a.kept_offsets,
                  a.packed_offsets, a.kept_idx, a.capacity, a.evicted_sum, a.total_sum, a.bitmap,
                  a.bm_stride, a.mask);
    return CERTKV_OK;
  };
  const auto forms = [&](auto whole) -> certkv_status {
    constexpr bool W = decltype(whole)::value;
    if (a.evicted_sum)
      return a.mask ? launch(select_kernel<W, true, true>) : launch(select_kernel<W, true, false>);
    return a.mask ? launch(select_kernel<W, false, true>) : launch(select_kernel<W, false, false>);
  };
  return grid.x == (unsigned)(a.g.H * st.count) ? forms(std::true_type()) : forms(std::false_type());
}

}  // namespace certkv
