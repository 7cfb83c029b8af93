// Budget allocation (multiplier bisection + one-token repair) on gfx950.
//
// One workgroup per (layer, sequence).
//
// Bisection.  Each step needs, per head, the smallest b in [b_min, n-1]
// minimizing f(b) = fma(lambda, b, c(b)) in fp64 on the fp32 curve.  The scan
// is pruned exactly: for a run of ranks starting at b0 (clamped to b_min)
// with minimum cmin, every candidate has lambda*b + c(b) >= lambda*b0 + cmin,
// and round-to-nearest is monotone, so LB = fma(lambda, b0, cmin) <= f(b) on
// the run (the runs are the two 128-rank halves of each 256-rank block).  The block with the smallest bound is evaluated
// first (32 threads per head); every block whose (LB, b0) undercuts the best
// (f*, b*) lexicographically is then put on a candidate list and evaluated
// by the whole workgroup, one coalesced 256-wide row per block.  Blocks left
// out cannot hold the answer (ties favour smaller b), so the result equals the
// full scan.
//
// Repair.  Starting from b_h = b_h(lambda_hi), the method adds one token at a
// time to the head with the smallest marginal d_h(i) = c_h(i+1) - c_h(i)
// (ties: lowest head).  That greedy consumes the candidate increments in
// increasing order of the key (P_h(i), h, i), where P_h(i) is the running
// maximum of d_h over [b_h, i]: all increments keyed below a level are taken
// before any keyed at or above it, and within a level the lowest head runs
// first.  So the final budgets follow from the R-th smallest key, R = B_real -
// sum b_h: a bisection over the ordered bit patterns of fp64 keys finds it,
// counting per head with block-level running maxima (LDS) and one scan of the
// block where the running maximum crosses the threshold.
//
// Hull.  For any lambda >= 0 the smallest f lies on the lower convex hull of the
// points (b, c(b)), b >= b_min: a few hundred of them, because the curves are
// noisy.  So the points that can never be an argmin are dropped first: p
// between a and c is dropped if it lies above their chord by more than the
// rounding of f can hide (hull_above), which leaves every f of the argmin and
// of its ties in place.  Two kernels filter (chunks of 2 or 8 blocks, then
// a unit's chunks) and one workgroup per (layer, sequence) bisects over the
// remaining points in LDS.  Its repair finds the R-th smallest key by value
// among the block maxima and then in the few blocks where the running maxima
// rise past it.  The searches above remain for curves whose hull is large
// (convex without noise: tail masses; flat or linear ones) and for sizes beyond
// LDS: the hull kernel leaves those (layer, sequence)s to them.
// Block statistics and allocation, before and with the hull: one layer of 8
// heads at 32768 tokens 13 + 212 us and 14 + 17 + 47 us, eight ragged sequences
// 16 + 229 and 29 + 27 + 51, 32 layers at 131072 57 + 305 and 143 + 21 + 60; the
// full search's launch that follows finds nothing to do in 2 us.
#include <type_traits>

#include "stages.h"

namespace certkv {

constexpr int kAllocThreads = 1024;
constexpr int kAllocWaves = kAllocThreads / 64;
constexpr int kHeadGroup = kAllocThreads / 32;  // heads handled concurrently (32 threads each)
constexpr int kCandCap = 1024;    // candidate blocks evaluated per round
constexpr int kBlk = 256;          // ranks per pruning block
constexpr int kLdsItems = 8192;    // H * blocks handled from LDS
// Hull points kept of a chunk (of 2 or 8 blocks), joined for a unit, and of a
// unit; doubles of the hull kernel's LDS pool and its loaded blocks at most.
constexpr int kChunkList = 512;    // of a chunk's list while it is filtered
constexpr int kChunkCap = 128;
constexpr int kMergeCap = 8192;
constexpr int kUnitCap = 1024;
constexpr int kHullPool = 15360;
constexpr int kHullSlots = 64;
constexpr int kRepairWin = 64;     // cached curve values per head (fallback repair)
constexpr int kRcStride = kBlk + 4;  // a cached curve block of the repair search: kBlk + 1 values
// Bisection across several workgroups per (layer, sequence): up to kTreeLev
// levels per pass, one workgroup per node of the level tree.
constexpr int kTreeLev = 3;
constexpr int kTreeMax = (1 << kTreeLev) - 1;
constexpr int kSyncGroups = 256;   // (layer, sequence) groups of one such launch at most
// sync words: ticket, pad, one word per group (unused), then per group and
// pass parity the nodes' budget sums tagged with their pass ((pass + 1) << 48
// | sum, int64) and argmin vectors (64 heads)
constexpr size_t kSyncCnt = 2 + kSyncGroups;
constexpr size_t kSyncSum = kSyncCnt;
constexpr size_t kSyncArg = kSyncSum + (size_t)kSyncGroups * 2 * kTreeMax * 2;
constexpr size_t kSyncWords = kSyncArg + (size_t)kSyncGroups * 2 * kTreeMax * 64;

size_t alloc_sync_words() { return kSyncWords; }
size_t alloc_chunk_points() { return kChunkCap; }

// Lanes below this one among those set in `mask`.
__device__ __forceinline__ uint32_t count_below64(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// A curve value as the block statistics and the repair read it: unchanged
// when finite; NaN and +inf read as the largest finite float, -inf as its
// negative.  The bisection's candidate scans read the curves as they are (a
// NaN never wins a comparison), and a head left without an argmin starts the
// repair from b_min.  So with non-finite curves (a caller's, or from
// non-finite inputs) the budgets still lie in [b_min, n-1] and sum to B_real,
// meaningless as they are, and the status word reports the values.
__device__ __forceinline__ float cval(float x) {
  constexpr float kMax = 3.40282347e38f;  // the largest finite float
  return fmaxf(fminf(x, kMax), -kMax);
}

__device__ __forceinline__ bool lex_less(double f1, int b1, double f2, int b2) {
  return f1 < f2 || (f1 == f2 && b1 < b2);
}

struct BestFB {
  double f;
  int b;
};

// Minimum over each half-wave (lanes 0-31 and 32-63), in every lane of the
// half: DPP exchanges within rows of 16 lanes (lane ^ 1, lane ^ 2, then the
// mirrored lane within 8 and within 16: after the first steps the values are
// equal within the smaller groups, so a mirror pairs the groups as an xor
// would), then v_permlane16_swap pairs the two rows of each half.  Every lane
// of a half must be active.
__device__ __forceinline__ int half_min_i32(int x) {
  x = min(x, __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false));
  x = min(x, __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false));
  x = min(x, __builtin_amdgcn_update_dpp(x, x, 0x141, 0xF, 0xF, false));
  x = min(x, __builtin_amdgcn_update_dpp(x, x, 0x140, 0xF, 0xF, false));
  const auto r = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)x, false, false);
  return min((int)r[0], (int)r[1]);
}

// The same minimum for floats (no NaN among the values).
__device__ __forceinline__ float half_min_f32(float x) {
  x = fminf(x, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), 0xB1, 0xF, 0xF, false)));
  x = fminf(x, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), 0x4E, 0xF, 0xF, false)));
  x = fminf(x, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), 0x141, 0xF, 0xF, false)));
  x = fminf(x, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), 0x140, 0xF, 0xF, false)));
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fminf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Lexicographic (f, b) minimum reductions, carrying a float c of the winning
// lane (the order is total on (f, b), so the result does not depend on the
// pairing).  The exchanges are those of half_min_i32, plus v_permlane32_swap
// for the whole wave; every lane of the reduced group must be active.
__device__ __forceinline__ void lex_take(double& f, int& b, float& c, double fo, int bo, float co) {
  if (lex_less(fo, bo, f, b)) {
    f = fo;
    b = bo;
    c = co;
  }
}

template <int CTL>
__device__ __forceinline__ void lex_dpp(double& f, int& b, float& c) {
  const uint64_t u = (uint64_t)__double_as_longlong(f);
  const int lo = __builtin_amdgcn_update_dpp((int)(uint32_t)u, (int)(uint32_t)u, CTL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(u >> 32), (int)(uint32_t)(u >> 32), CTL,
                                             0xF, 0xF, false);
  const int bo = __builtin_amdgcn_update_dpp(b, b, CTL, 0xF, 0xF, false);
  const int co = __builtin_amdgcn_update_dpp(__float_as_int(c), __float_as_int(c), CTL, 0xF, 0xF, false);
  const double fo = __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
  lex_take(f, b, c, fo, bo, __int_as_float(co));
}

// One exchange between the pairs of 16-lane rows of each half (W = 16) or
// between the halves (W = 32): both candidates arrive in every lane.
template <int W>
__device__ __forceinline__ void lex_swap(double& f, int& b, float& c) {
  const uint64_t u = (uint64_t)__double_as_longlong(f);
  const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
  const uint32_t bu = (uint32_t)b, cu = __float_as_uint(c);
  auto sw = [](uint32_t x) {
    if constexpr (W == 16)
      return __builtin_amdgcn_permlane16_swap(x, x, false, false);
    else
      return __builtin_amdgcn_permlane32_swap(x, x, false, false);
  };
  const auto rl = sw(lo), rh = sw(hi), rb = sw(bu), rc = sw(cu);
  f = __longlong_as_double((long long)(((uint64_t)rh[0] << 32) | rl[0]));
  b = (int)rb[0];
  c = __uint_as_float(rc[0]);
  lex_take(f, b, c, __longlong_as_double((long long)(((uint64_t)rh[1] << 32) | rl[1])), (int)rb[1],
           __uint_as_float(rc[1]));
}

// over `WIDTH` lanes: 32 (each half-wave) or 64 (the wave)
template <int WIDTH>
__device__ __forceinline__ void lexmin_fbc(double& f, int& b, float& c) {
  lex_dpp<0xB1>(f, b, c);   // lane ^ 1
  lex_dpp<0x4E>(f, b, c);   // lane ^ 2
  lex_dpp<0x141>(f, b, c);  // mirrored within 8
  lex_dpp<0x140>(f, b, c);  // mirrored within 16
  lex_swap<16>(f, b, c);
  if constexpr (WIDTH == 64) lex_swap<32>(f, b, c);
}

__device__ __forceinline__ BestFB half_wave_min(double f, int b) {
  float c = 0.f;
  lexmin_fbc<32>(f, b, c);
  return BestFB{f, b};
}

__device__ __forceinline__ BestFB wave_lexmin(double f, int b) {
  float c = 0.f;
  lexmin_fbc<64>(f, b, c);
  return BestFB{f, b};
}

// Minimum of a double, and sum of an int, over the wave, in every lane.
__device__ __forceinline__ double wave_min_f64(double x) {
  auto join = [](uint32_t lo, uint32_t hi) {
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
  };
  auto dpp = [&](auto ctl) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const int lo = (int)(uint32_t)u, hi = (int)(uint32_t)(u >> 32);
    x = fmin(x, join((uint32_t)__builtin_amdgcn_update_dpp(lo, lo, decltype(ctl)::value, 0xF, 0xF, false),
                     (uint32_t)__builtin_amdgcn_update_dpp(hi, hi, decltype(ctl)::value, 0xF, 0xF, false)));
  };
  dpp(std::integral_constant<int, 0xB1>());
  dpp(std::integral_constant<int, 0x4E>());
  dpp(std::integral_constant<int, 0x141>());
  dpp(std::integral_constant<int, 0x140>());
  {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    x = fmin(join(a[0], b[0]), join(a[1], b[1]));
  }
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
  const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  return fmin(join(a[0], b[0]), join(a[1], b[1]));
}
__device__ __forceinline__ int wave_sum_i32(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x140, 0xF, 0xF, false);
  const auto a = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)x, false, false);
  x = (int)a[0] + (int)a[1];
  const auto b = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
  return (int)b[0] + (int)b[1];
}

// Monotone map between fp64 values and unsigned keys (total order of doubles).
__device__ __forceinline__ uint64_t dkey(double x) {
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  return (u & 0x8000000000000000ull) ? ~u : (u | 0x8000000000000000ull);
}
__device__ __forceinline__ double dval(uint64_t k) {
  const uint64_t u = (k & 0x8000000000000000ull) ? (k & 0x7fffffffffffffffull) : ~k;
  return __longlong_as_double((long long)u);
}

// Per-block statistics of the curves: minimum of c over each 128-rank half of
// each 256-rank block (+inf where a half is past the end), maximum of c over
// the block, the smallest position holding the block minimum, and the
// maximum marginal d(i) = c(i+1) - c(i) (fp64) over the i of the block with
// i <= n-2.  One wave per NB consecutive blocks (a chunk), the loads of all of
// them in flight at once (positions clamped into the segment, masked where
// used); lane L covers positions 4L..4L+3 of a block (lanes 0-31 the first
// half), and the wave reductions are DPP and lane-row exchanges.

template <typename T, typename F>
__device__ __forceinline__ T wave_reduce_dpp(T x, F op) {
  static_assert(sizeof(T) == 4, "32-bit values");
  auto dpp = [&](auto ctl) {
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, x), __builtin_bit_cast(int, x),
                                                             decltype(ctl)::value, 0xF, 0xF, false));
  };
  x = op(x, dpp(std::integral_constant<int, 0xB1>()));
  x = op(x, dpp(std::integral_constant<int, 0x4E>()));
  x = op(x, dpp(std::integral_constant<int, 0x141>()));
  x = op(x, dpp(std::integral_constant<int, 0x140>()));
  // (the swap results are read into scalars before the bit casts: a bit cast
  // applied to a subscripted element of the result vector compiled to the
  // first element for both subscripts)
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const auto r16 = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const uint32_t a0 = r16[0], a1 = r16[1];
  x = op(__builtin_bit_cast(T, a0), __builtin_bit_cast(T, a1));
  const uint32_t v = __builtin_bit_cast(uint32_t, x);
  const auto r32 = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  const uint32_t b0 = r32[0], b1 = r32[1];
  return op(__builtin_bit_cast(T, b0), __builtin_bit_cast(T, b1));
}

// Whether point p = (b, c) lies above the chord of the points a and d around it
// by more than rounding can hide, so that it is never an argmin.  Let s be the
// chord's fall per rank and h the height above it.  For lambda >= s, f(p) - f(a)
// = (lambda - s)(p - a) + h, and for lambda < s, f(p) - f(d) = (s - lambda)(d - p)
// + h, both exactly; each f carries one rounding, u = 2^-53 of its size, and the
// size at lambda = s, where the difference is smallest, is at most max(s, 0) p +
// |c|.  So h above 2 u (max(s, 0) p + |c_p| + |c_a| + |c_d|) decides for every
// lambda; the factor taken, 36 u, also covers the rounding of h here.  (A
// non-finite value is never above anything, and nothing is above it.)
__device__ __forceinline__ bool hull_above(int ba, float ca, int bp, float cp, int bd, float cd) {
  const double da = (double)(bp - ba), dd = (double)(bd - bp);
  const double xa = (double)ca, xp = (double)cp, xd = (double)cd;
  const double rise = (xp - xa) * dd + (xp - xd) * da;  // h (d - a)
  const double size = (fabs(xa) + fabs(xp) + fabs(xd)) * (da + dd) + fmax(xa - xd, 0.0) * (double)bp;
  return rise > 4e-15 * size;
}

// Drop the points of an ascending list above the chord of their neighbours,
// until none is left or `rounds` are done; the first and the last stay.  One
// wave, 256 points at a time (four of a lane's in flight); the list is compacted
// in place (a batch writes no place that a later one still reads as another
// point).  Points dropped together may be each other's neighbours: each is
// beaten at every lambda by some point of the list, and the argmin by none.
__device__ __forceinline__ int hull_filter(uint2* pts, int m, int rounds, int lane) {
  constexpr int Q = 4;
  for (int it = 0; it < rounds && m > 2; ++it) {
    int out = 0;
    for (int r0 = 0; r0 < m; r0 += 64 * Q) {
      uint2 a[Q], x[Q], d[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int i = r0 + 64 * q + lane;
        a[q] = pts[min(max(i - 1, 0), m - 1)];
        x[q] = pts[min(i, m - 1)];
        d[q] = pts[min(i + 1, m - 1)];
      }
      __asm__ volatile("" ::: "memory");  // a wave's LDS accesses execute in order
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int i = r0 + 64 * q + lane;
        if (r0 + 64 * q >= m) break;
        const bool keep = i < m && (i == 0 || i == m - 1 ||
                                    !hull_above((int)a[q].x, __uint_as_float(a[q].y), (int)x[q].x,
                                                __uint_as_float(x[q].y), (int)d[q].x,
                                                __uint_as_float(d[q].y)));
        const uint64_t bal = __ballot(keep);
        if (keep) pts[out + (int)count_below64(bal)] = x[q];
        out += (int)__popcll(bal);
      }
      __asm__ volatile("" ::: "memory");
    }
    if (out == m) break;
    m = out;
  }
  return m;
}

// Chunks of nb blocks of a unit of n ranks, and the first one of a unit's in the
// chunks' arrays (one entry per chunk of the launch).
__device__ __forceinline__ int hull_chunks(int n, int nb) {
  return ((n + kBlk - 1) / kBlk + nb - 1) / nb;
}
__device__ __forceinline__ int64_t hull_base(const Geo& g, const SeqTab& st, int l, int bl, int h,
                                             int nb) {
  return part_base(g, st, l, bl, h, [&](int i) { return hull_chunks(st.len[i], nb); });
}

template <bool HULL, int NB>
__global__ __launch_bounds__(256) void curve_blockstats_kernel(Geo g, SeqTab st, int32_t nblk_max,
                                                               const float* __restrict__ curves,
                                                               float* __restrict__ cmin,
                                                               float* __restrict__ cmaxb,
                                                               int32_t* __restrict__ cpos,
                                                               double* __restrict__ dmax,
                                                               int32_t* __restrict__ sync, int32_t nsync,
                                                               uint2* __restrict__ hull_pts,
                                                               int32_t* __restrict__ hull_cnt) {
  __shared__ __align__(16) uint2 hlist[HULL ? 4 : 1][HULL ? kChunkList : 1];
  // the allocation's exchange words (ticket, tagged sums) start at zero: the
  // first workgroup clears them for the allocation kernel launched next
  if (sync && blockIdx.x == 0 && blockIdx.y == 0)
    for (int i = threadIdx.x; i < nsync; i += 256) sync[i] = 0;
  const int per_unit = (nblk_max + 4 * NB - 1) / (4 * NB);
  const int wb = blockIdx.x % per_unit;
  const int hb = blockIdx.x / per_unit;
  const int h = hb % g.H;
  const int bl = hb / g.H;
  const int l = blockIdx.y;
  if (bl >= st.count) return;
  const int n = st.len[bl];
  const int nblk = (n + kBlk - 1) / kBlk;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int k0 = (wb * 4 + wave) * NB;
  if (k0 >= nblk) return;
  const int64_t u = unit_index(g, l, st.first + bl, h);
  const float* ch = curves + lht_base(g, l, h, st.start[bl]);
  float c[NB][5];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int i0 = (k0 + j) * kBlk + lane * 4;
#pragma unroll
    for (int e = 0; e < 5; ++e) c[j][e] = ch[min(i0 + e, n - 1)];
  }
  // a caller's non-finite curve values: reported, then read as cval() reads them
  bool bad = false;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
#pragma unroll
    for (int e = 0; e < 5; ++e) {
      bad |= !isfinite(c[j][e]);
      c[j][e] = cval(c[j][e]);
    }
  }
  if (__ballot(bad) != 0ull && lane == 0) report_nonfinite(g);
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int k = k0 + j;
    if (k >= nblk) break;
    const int i0 = k * kBlk + lane * 4;
    float mn = INFINITY, mx = -INFINITY;
    int pmn = 0x7fffffff;
    double dm = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (i0 + e < n) {
        if (c[j][e] < mn) {
          mn = c[j][e];
          pmn = i0 + e;
        }
        mx = fmaxf(mx, c[j][e]);
      }
      if (i0 + e <= n - 2) dm = fmax(dm, (double)c[j][e + 1] - (double)c[j][e]);
    }
    const float mhalf = half_min_f32(mn);
    // (min c, smallest position): the lexicographic minimum of (c, position)
    // (min c, smallest position): the smallest position holding the minimum
    const float mnw = wave_reduce_dpp(mn, [](float a, float b) { return fminf(a, b); });
    const int pw = wave_reduce_dpp(mn == mnw ? pmn : 0x7fffffff, [](int a, int b) { return min(a, b); });
    mx = wave_reduce_dpp(mx, [](float a, float b) { return fmaxf(a, b); });
    dm = wave_max(dm);
    if ((lane & 31) == 0) cmin[(u * nblk_max + k) * 2 + (lane >> 5)] = mhalf;
    if (lane == 0) {
      cmaxb[u * nblk_max + k] = mx;
      cpos[u * nblk_max + k] = pw;
      dmax[u * nblk_max + k] = dm;
    }
  }
  if constexpr (HULL) {
    // The chunk's hull points.  An anchor per block, the point lowest against
    // the chunk's mean fall (any point is a valid anchor), and the chunk's
    // first and last points: nearly all the others lie above the chords between
    // consecutive anchors.  The rest go to the wave's list, filtered as it
    // fills and at the end.
    const int bmin = st.b_min[bl];
    const int c_lo = max(k0 * kBlk, bmin), c_hi = min((k0 + NB) * kBlk, n) - 1;
    const bool over0 = __ballot(bad) != 0ull;
    const int64_t ch_i = hull_base(g, st, l, bl, h, NB) + k0 / NB;
    if (c_lo > c_hi || over0) {
      if (lane == 0) hull_cnt[ch_i] = over0 ? -1 : 0;
      return;
    }
    const float f_lo = cval(ch[c_lo]), f_hi = cval(ch[c_hi]);
    const float fall = c_hi > c_lo ? (f_lo - f_hi) / (float)(c_hi - c_lo) : 0.f;
    int tb[NB];    // each block's anchor (-1: no point of the block is in range)
    float tc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int i0 = (k0 + j) * kBlk + lane * 4;
      float best = INFINITY, bc = 0.f;
      int be = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool in = i0 + e >= c_lo && i0 + e <= c_hi;
        const float v = in ? fmaf(fall, (float)(i0 + e - c_lo), c[j][e]) : INFINITY;
        if (v < best) {
          best = v;
          bc = c[j][e];
          be = e;
        }
      }
      const float mn = wave_reduce_dpp(best, [](float x, float y) { return fminf(x, y); });
      const uint64_t at = __ballot(best == mn && best < INFINITY);
      tb[j] = -1;
      tc[j] = 0.f;
      if (at) {
        const int src = (int)__builtin_ctzll(at);
        tb[j] = (k0 + j) * kBlk + src * 4 + __builtin_amdgcn_readlane(be, src);
        tc[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bc), src));
      }
    }
    uint2* list = hlist[wave];
    int m = 0;
    bool over = false;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (tb[j] < 0) continue;
      const int i0 = (k0 + j) * kBlk + lane * 4;
      const bool hp = j > 0 && tb[j > 0 ? j - 1 : 0] >= 0;
      const bool hn = j + 1 < NB && tb[j + 1 < NB ? j + 1 : j] >= 0;
      const int pb = hp ? tb[j > 0 ? j - 1 : 0] : c_lo;
      const float pc = hp ? tc[j > 0 ? j - 1 : 0] : f_lo;
      const int nb = hn ? tb[j + 1 < NB ? j + 1 : j] : c_hi;
      const float nc = hn ? tc[j + 1 < NB ? j + 1 : j] : f_hi;
      // the chord on the lane's side of the anchor; with the anchor among its
      // points, or none on that side, the lane keeps them all (hull_above's
      // bound, doubled)
      const bool left = i0 + 3 < tb[j], right = i0 > tb[j];
      const int ba = left ? pb : tb[j], bd = left ? tb[j] : nb;
      const double xa = (double)(left ? pc : tc[j]), xd = (double)(left ? tc[j] : nc);
      const double slope = (xd - xa) / (double)(bd - ba);
      const double t0 = 8e-15 * (fabs(xa) + fabs(xd) + fmax(-slope, 0.0) * (double)bd);
      const double y0 = fma(slope, (double)(i0 - ba), xa);
      bool keep[4];
      uint64_t bal[4];
      int below = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = i0 + e;
        const double x = (double)c[j][e];
        const double rise = x - fma(slope, (double)e, y0);
        const bool drop = (left || right) && i > c_lo && i < c_hi && rise > fma(8e-15, fabs(x), t0);
        keep[e] = i >= c_lo && i <= c_hi && !drop;
        bal[e] = __ballot(keep[e]);
        below += (int)count_below64(bal[e]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (keep[e]) list[m + below++] = make_uint2((uint32_t)(i0 + e), __float_as_uint(c[j][e]));
#pragma unroll
      for (int e = 0; e < 4; ++e) m += (int)__popcll(bal[e]);
      __asm__ volatile("" ::: "memory");
      if (m > kChunkList - kBlk) m = hull_filter(list, m, 6, lane);
      if (m > kChunkList - kBlk) {  // no room for another block: left to the full search
        over = true;
        m = 0;
      }
    }
    m = hull_filter(list, m, 6, lane);
    over = over || m > kChunkCap;
    if (lane == 0) hull_cnt[ch_i] = over ? -1 : m;
    if (!over)
      for (int i = lane; i < m; i += 64) hull_pts[ch_i * kChunkCap + i] = list[i];
  }
}

// A unit's chunk lists joined, filtered again and written over the first of them,
// and its largest curve value.
// Count -1: a chunk or the unit has too many points.
constexpr int kMergeThreads = 256;
__global__ __launch_bounds__(kMergeThreads) void hull_merge_kernel(
    Geo g, SeqTab st, int32_t nblk_max, int32_t nb, const float* __restrict__ cmaxb,
    uint2* __restrict__ hull_pts, const int32_t* __restrict__ hull_cnt,
    int32_t* __restrict__ unit_cnt, float* __restrict__ unit_max) {
  __shared__ __align__(16) uint2 list[kMergeCap];
  __shared__ int32_t off[kLdsItems / 2 + 1];  // where each chunk's points go
  __shared__ float mx_s[kMergeThreads / 64];
  const int h = blockIdx.x % g.H;
  const int bl = blockIdx.x / g.H;
  const int l = blockIdx.y;
  if (bl >= st.count) return;
  const int n = st.len[bl];
  const int64_t u = unit_index(g, l, st.first + bl, h);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nblk = (n + kBlk - 1) / kBlk;
  const int nchunk = hull_chunks(n, nb);  // <= kLdsItems / 2
  const int64_t ch0 = hull_base(g, st, l, bl, h, nb);
  float mx = -INFINITY;
#pragma unroll 4
  for (int k = tid; k < nblk; k += kMergeThreads) mx = fmaxf(mx, cmaxb[u * nblk_max + k]);
  mx = wave_max(mx);
  if (lane == 0) mx_s[wave] = mx;
  if (wave == 0) {
    int run = 0;
    for (int q0 = 0; q0 < nchunk; q0 += 64) {
      int c = q0 + lane < nchunk ? hull_cnt[ch0 + q0 + lane] : 0;
      if (__ballot(c < 0) != 0ull) c = kMergeCap + 1;  // a chunk overflowed: so does the unit
      int incl = c;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
      }
      if (q0 + lane < nchunk) off[q0 + lane + 1] = run + incl;
      run += __shfl(incl, 63, 64);
    }
    if (lane == 0) off[0] = 0;
  }
  __syncthreads();
  int m = off[nchunk];
  const bool fits = m <= kMergeCap;
  if (fits) {
    // sixteen chunks of a wave in flight (64 of a chunk's points per load)
    constexpr int Q = 16, W = kMergeThreads / 64;
    for (int q0 = wave; q0 < nchunk; q0 += Q * W) {
      uint2 x[Q];
#pragma unroll
      for (int j = 0; j < Q; ++j) {
        const int q = min(q0 + j * W, nchunk - 1);
        x[j] = hull_pts[(ch0 + q) * kChunkCap + lane];
      }
#pragma unroll
      for (int j = 0; j < Q; ++j) {
        const int q = q0 + j * W;
        if (q < nchunk && lane < off[q + 1] - off[q]) list[off[q] + lane] = x[j];
      }
      for (int j = 0; j < Q; ++j) {  // the few chunks of more than 64
        const int q = q0 + j * W;
        if (q < nchunk)
          for (int i = 64 + lane; i < off[q + 1] - off[q]; i += 64)
            list[off[q] + i] = hull_pts[(ch0 + q) * kChunkCap + i];
      }
    }
  }
  __syncthreads();
  if (wave != 0) return;
  if (fits) m = hull_filter(list, m, 6, lane);
  const bool over = !fits || m > kUnitCap;
  if (!over)
    for (int i = lane; i < m; i += 64) hull_pts[ch0 * kChunkCap + i] = list[i];
  if (lane == 0) {
    unit_cnt[u] = over ? -1 : m;
    for (int w = 0; w < kMergeThreads / 64; ++w) mx = fmaxf(mx, mx_s[w]);
    unit_max[u] = mx;
  }
}

// The allocation of one (layer, sequence) over its heads' hull points.  Bound
// by its chain of about 40 + 10 dependent steps, each an LDS round trip and a
// barrier.
__global__ __launch_bounds__(kAllocThreads) void allocate_hull_kernel(
    Geo g, SeqTab st, const float* __restrict__ curves, const double* __restrict__ dmax,
    int32_t nblk_max, int32_t nb, int32_t steps, const uint2* __restrict__ hull_pts,
    const int32_t* __restrict__ unit_cnt, const float* __restrict__ unit_max,
    int32_t* __restrict__ budgets, int64_t* __restrict__ stats, int32_t* __restrict__ done) {
  // hull points; then block running maxima, and blocks of running maxima
  __shared__ __align__(16) double pool[kHullPool];
  __shared__ int16_t slot_of[kLdsItems];  // block -> loaded block (Stage B), by h nblk + k
  __shared__ int32_t cnt_s[64], off_s[65];
  __shared__ int32_t bh_s[64];
  __shared__ double steep_s[64], size_s[64];
  __shared__ int32_t s_s[64], ks_s[64], ke_s[64];  // start, its block, end of the head's blocks
  __shared__ int32_t il[2][kHullSlots], ir[2][kHullSlots];  // candidate intervals per list
  __shared__ int32_t pcount[2][kAllocThreads / 2];          // counts of the pivots
  __shared__ uint64_t best_s[2], fail_s[2];
  __shared__ int32_t open_s[2];
  __shared__ int32_t nslot, sh_s[kHullSlots], sk_s[kHullSlots], after_s[kHullSlots];
  __shared__ int32_t lt_s[64], le_s[64];
  const int bl = blockIdx.x, l = blockIdx.y;
  const int b = st.first + bl;
  const int n = st.len[bl];
  const int64_t tok0 = st.start[bl];
  const int64_t B_real = st.b_real[bl];
  const int bmin = st.b_min[bl];
  const int H = g.H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nblk = (n + kBlk - 1) / kBlk;
  const int64_t u0 = unit_index(g, l, b, 0);
  const uint64_t t_start = wall_clock64();
  int32_t* flag = done + (int64_t)l * g.B + b;

  if (tid < H) cnt_s[tid] = unit_cnt[u0 + tid];
  __syncthreads();
  int total = 0;
  bool ok = H * nblk <= kLdsItems;
  float cmf = 0.f;
  for (int h = 0; h < H; ++h) {
    if (tid == 0) off_s[h] = total;
    if (cnt_s[h] < 0) ok = false;
    total += max(cnt_s[h], 0);
    cmf = fmaxf(cmf, unit_max[u0 + h]);
  }
  ok = ok && total <= kHullPool;
  if (!ok) {  // (the same for every thread)
    if (tid == 0) *flag = 0;
    return;
  }
  uint2* pts = reinterpret_cast<uint2*>(pool);
  __syncthreads();
  const int64_t ch0 = hull_base(g, st, l, bl, 0, nb), per_head = (int64_t)hull_chunks(n, nb) * g.L;
  for (int h = wave; h < H; h += kAllocWaves) {
    const int m = cnt_s[h];
    const uint2* p = hull_pts + (ch0 + h * per_head) * kChunkCap;
#pragma unroll 4
    for (int i = lane; i < m; i += 64) pts[off_s[h] + i] = p[i];
  }
  __syncthreads();

  // Per head, the steepest chord from its first point (b_min) and the largest
  // size of a value.
  for (int h = wave; h < H; h += kAllocWaves) {
    const uint2* p = pts + off_s[h];
    const int m = cnt_s[h];
    const double x0 = (double)__uint_as_float(p[0].y), b0 = (double)(int)p[0].x;
    double steep = -INFINITY, size = fabs(x0);
    for (int i = 1 + lane; i < m; i += 64) {
      const double x = (double)__uint_as_float(p[i].y);
      steep = fmax(steep, (x0 - x) / ((double)(int)p[i].x - b0));
      size = fmax(size, fabs(x));
    }
    steep = -wave_min_f64(-steep);
    size = -wave_min_f64(-size);
    if (lane == 0) {
      steep_s[h] = steep;
      size_s[h] = size;
    }
  }
  __syncthreads();
  // The bisection, by one wave: no step has a barrier.  Each head has 64 / G
  // lanes, which share out the points between its argmins at hi and at lo.
  if (wave == 0) {
    int G = 1, lph = 64;
    while (G < H) {
      G *= 2;
      lph /= 2;
    }
    const int h = lane / lph, sub = lane - h * lph;
    const bool act = h < H;
    const uint2* p = pts + off_s[act ? h : 0];
    const int m = act ? cnt_s[h] : 0;
    double steep = -INFINITY, size = 0.0;
    for (int x = 0; x < H; ++x) {
      steep = fmax(steep, steep_s[x]);
      size = fmax(size, size_s[x]);
    }
    // argmin over the points [ia, ib] of the lane's head: its b, and its index
    auto argmin = [&](double lam, int ia, int ib, int& idx) -> int {
      double f = INFINITY;
      int bb = 0x7fffffff, at = ia;
#pragma unroll 4
      for (int i = ia + sub; i <= ib; i += lph) {
        const uint2 x = p[i];
        const double v = fma(lam, (double)(int)x.x, (double)__uint_as_float(x.y));
        if (v < f) {
          f = v;
          bb = (int)x.x;
          at = i;
        }
      }
      float c = __int_as_float(at);
      if (lph >= 2) lex_dpp<0xB1>(f, bb, c);
      if (lph >= 4) lex_dpp<0x4E>(f, bb, c);
      if (lph >= 8) lex_dpp<0x141>(f, bb, c);
      if (lph >= 16) lex_dpp<0x140>(f, bb, c);
      if (lph >= 32) lex_swap<16>(f, bb, c);
      if (lph >= 64) lex_swap<32>(f, bb, c);
      idx = __float_as_int(c);
      return bb;
    };
    double lo = 0.0, hi = 2.0 * (double)cmf + 1.0;
    int i_lo = m - 1, i_hi = 0;  // the argmins lie between these points
    bool have = false;
    int bh = bmin;
    int t = 0;
    // At twice the steepest chord every f(p) exceeds f(b_min) by lambda / 2 per
    // rank at least, far more than rounding: every head's argmin is b_min, and
    // H b_min <= B_real lowers hi.
    const double far = fmax(2.0 * steep, 1e-12 * size);
    for (; t < steps; ++t) {
      const double lam = (lo + hi) / 2.0;
      if (!(lam > far)) break;
      hi = lam;
      have = true;
    }
    for (; t < steps; ++t) {
      const double lam = (lo + hi) / 2.0;
      int idx;
      const int bb = argmin(lam, i_hi, i_lo, idx);
      // (sums of int32 argmins: H <= 64 heads of n < 2^31, two halves)
      const int mine = act && sub == 0 ? bb : 0;
      const int64_t sum = ((int64_t)wave_sum_i32(mine >> 16) << 16) + wave_sum_i32(mine & 0xffff);
      if (sum > B_real)
        lo = lam;
      else {
        hi = lam;
        have = true;
        bh = bb;
      }
      // A larger lambda has its argmin at the same b or below.  For two
      // multipliers a distance w apart and points a rank apart, the exact
      // difference of the f's grows by w at least, so the computed argmins keep
      // that order while w is well above the f's roundings, 2^-53 of their size.
      const double w = (hi - lo) / 2.0;
      if (w > 1e-14 * (hi * (double)n + size)) {
        if (sum > B_real)
          i_lo = idx;
        else
          i_hi = idx;
      } else {
        i_lo = m - 1;
        i_hi = 0;
      }
    }
    if (!have) {
      int idx;
      bh = argmin(hi, 0, m - 1, idx);
    }
    if (act && sub == 0) bh_s[h] = bh;
  }
  __syncthreads();
  const int32_t bh = tid < H ? bh_s[tid] : 0;
  const uint64_t t_bisect = wall_clock64();
  const int kmax = (n - 2) / kBlk;  // last block holding an increment i <= n-2
  if (tid < H) {
    s_s[tid] = bh;
    ks_s[tid] = bh / kBlk;
    ke_s[tid] = bh > n - 2 ? bh / kBlk : kmax + 1;
  }
  __syncthreads();
  int64_t sum0 = 0;
  for (int h = 0; h < H; ++h) sum0 += s_s[h];
  const int64_t R = B_real - sum0;
  if (R < 0) {
    if (tid == 0) *flag = 0;
    return;
  }
  if (R > 0) {
    // Stage A.  Running maxima of the marginals at the ends of the blocks, as
    // in the search of allocate_kernel.
    double* pbm = pool;
#pragma unroll 4
    for (int i = tid; i < H * nblk; i += kAllocThreads) {
      const int h = i / nblk, k = i - h * nblk;
      pbm[i] = dmax[(u0 + h) * nblk_max + k];
    }
    __syncthreads();
    for (int h = wave; h < H; h += kAllocWaves) {
      const float* ch = curves + lht_base(g, l, h, tok0);
      const int s = s_s[h], ks = ks_s[h], ke = ke_s[h];
      double dm = -INFINITY;
      if (ke > ks) {
        const int e1 = min(ks * kBlk + kBlk - 1, n - 2);
        for (int i = s + lane; i <= e1; i += 64)
          dm = fmax(dm, (double)cval(ch[i + 1]) - (double)cval(ch[i]));
      }
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) dm = fmax(dm, __shfl_xor(dm, m, 64));
      double* ph = pbm + h * nblk;
      double carry = -INFINITY;
      for (int k0 = 0; k0 < nblk; k0 += 64) {
        const int k = k0 + lane;
        double x = -INFINITY;
        if (k >= ks && k < ke) x = k == ks ? dm : ph[k];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const double y = __shfl_up(x, o, 64);
          if (lane >= o) x = fmax(x, y);
        }
        x = fmax(x, carry);
        if (k < nblk) ph[k] = x;
        carry = __shfl(x, 63, 64);
      }
    }
    // increments of head h in its blocks below k
    auto below = [&](int h, int k) -> int {
      return k <= ks_s[h] ? 0 : min(k * kBlk, n - 1) - s_s[h];
    };
    // first block of head h in [a, e) whose running maximum is above v, and
    // not below v
    auto first_above = [&](int h, int a, int e, double v) {
      const double* ph = pbm + h * nblk;
      while (a < e) {
        const int mid = (a + e) >> 1;
        if (ph[mid] > v) e = mid;
        else a = mid + 1;
      }
      return a;
    };
    auto first_not_below = [&](int h, int a, int e, double v) {
      const double* ph = pbm + h * nblk;
      while (a < e) {
        const int mid = (a + e) >> 1;
        if (ph[mid] >= v) e = mid;
        else a = mid + 1;
      }
      return a;
    };
    // The smallest block maximum v such that the increments certainly keyed at
    // or below it (whole blocks, q = 0) or possibly so (the crossing blocks
    // too, q = 1) reach R: the R-th key T lies in (anything below the second,
    // the first].  Pivots at even steps of the candidates, a thread per (pivot,
    // head), until every candidate has been tried or the rest are equal.
    int G = 1;
    while (G < H) G *= 2;
    const int NP = kAllocThreads / 2 / G;  // pivots of each question
    if (tid < 2 * H) {
      const int q = tid / H, h = tid - q * H;
      il[q][h] = ks_s[h];
      ir[q][h] = ke_s[h];
    }
    if (tid < 2) {
      best_s[tid] = ~0ull;
      fail_s[tid] = 0ull;
      open_s[tid] = 1;
    }
    __syncthreads();
    const int q = tid >> 9, pv = (tid & 511) / G, hq = (tid & 511) % G;
    int rounds = 0;
    while (open_s[0] | open_s[1]) {
      if (++rounds > 64) {  // (not reached: every round tries a pivot)
        if (tid == 0) *flag = 0;
        return;
      }
      const bool open = open_s[q] != 0;
      int cnt = 0;
      for (int h = 0; h < H; ++h) cnt += ir[q][h] - il[q][h];
      const int stride = (cnt + NP - 1) / NP;
      (&pcount[0][0])[tid] = 0;
      __syncthreads();
      int idx = pv * stride;
      const bool live = open && idx < cnt;
      double v = 0.0;
      if (live) {
        int h = 0;
        while (idx >= ir[q][h] - il[q][h]) {
          idx -= ir[q][h] - il[q][h];
          ++h;
        }
        v = pbm[h * nblk + il[q][h] + idx];
        if (hq < H) {
          const int k = first_above(hq, ks_s[hq], ke_s[hq], v);
          atomicAdd(&pcount[q][pv], below(hq, q == 0 ? k : min(k + 1, ke_s[hq])));
        }
      }
      __syncthreads();
      if (live && hq == 0) {
        if ((int64_t)(uint32_t)pcount[q][pv] >= R)
          atomicMin((unsigned long long*)&best_s[q], (unsigned long long)dkey(v));
        else
          atomicMax((unsigned long long*)&fail_s[q], (unsigned long long)dkey(v));
      }
      __syncthreads();
      // what is left: above every failure and below the best (whose equals, a
      // plateau of running maxima, would only take up pivots)
      if (open && (tid & 511) < H) {
        const int h = tid & 511;
        int a = il[q][h], e = ir[q][h];
        if (fail_s[q] != 0ull) a = first_above(h, a, e, dval(fail_s[q]));
        if (best_s[q] != ~0ull) e = first_not_below(h, a, e, dval(best_s[q]));
        il[q][h] = a;
        ir[q][h] = e;
      }
      __syncthreads();
      if ((tid & 511) == 0 && open) {
        bool more = false;
        if (stride > 1)
          for (int h = 0; h < H; ++h)
            if (il[q][h] < ir[q][h]) more = true;
        open_s[q] = more ? 1 : 0;
      }
      __syncthreads();
    }
    const double p_hi = dval(best_s[0]), p_lo = dval(best_s[1]);
    // Stage B.  The blocks that can hold T: those in which the running maximum
    // rises, from the first that reaches p_lo to the one that passes p_hi.
    // (Blocks in which it stands still hold the value it came in with.)
    if (tid < H) {
      const int a = first_not_below(tid, ks_s[tid], ke_s[tid], p_lo);
      il[0][tid] = a;
      ir[0][tid] = min(first_above(tid, a, ke_s[tid], p_hi) + 1, ke_s[tid]);
      lt_s[tid] = below(tid, a);  // all of them keyed below T
    }
    if (tid == 0) nslot = 0;
    __syncthreads();
    for (int i = tid; i < H * nblk; i += kAllocThreads) {
      const int h = i / nblk, k = i - h * nblk;
      int sl = -1;
      if (k >= il[0][h] && k < ir[0][h] && (k == ks_s[h] || pbm[i] > pbm[i - 1])) {
        sl = atomicAdd(&nslot, 1);
        if (sl < kHullSlots) {
          sh_s[sl] = h;
          sk_s[sl] = k;
        }
      }
      slot_of[i] = (int16_t)min(sl, kHullSlots);
    }
    __syncthreads();
    const int ns = nslot;
    if (ns < 1 || ns > kHullSlots || H * nblk + ns * kBlk > kHullPool) {
      if (tid == 0) *flag = 0;
      return;
    }
    double* blk = pool + H * nblk;  // running maxima of the loaded blocks
    for (int x = wave; x < ns; x += kAllocWaves) {
      const int h = sh_s[x], k = sk_s[x];
      const float* ch = curves + lht_base(g, l, h, tok0);
      float c[5];
#pragma unroll
      for (int e = 0; e < 5; ++e) c[e] = cval(ch[min(k * kBlk + lane * 4 + e, n - 1)]);
      double r[4], run = k > ks_s[h] ? pbm[h * nblk + k - 1] : -INFINITY;
      double mx = -INFINITY;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = k * kBlk + lane * 4 + e;
        const double d = i < s_s[h] ? -INFINITY
                         : i > n - 2 ? INFINITY  // past the last increment: never counted
                                     : (double)c[e + 1] - (double)c[e];
        mx = fmax(mx, d);
        r[e] = mx;
      }
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const double y = __shfl_up(mx, o, 64);
        if (lane >= o) mx = fmax(mx, y);
      }
      const double before = __shfl_up(mx, 1, 64);
      if (lane > 0) run = fmax(run, before);
#pragma unroll
      for (int e = 0; e < 4; ++e) blk[x * kBlk + lane * 4 + e] = fmax(run, r[e]);
      // increments of the still blocks after this one, up to the next loaded
      // one or the end of the range
      int k2 = k + 1;
      while (k2 < ir[0][h]) {
        const uint64_t stop = __ballot(k2 + lane >= ir[0][h] ||
                                       slot_of[min(h * nblk + k2 + lane, H * nblk - 1)] >= 0);
        if (stop) {
          k2 += (int)__builtin_ctzll(stop);
          break;
        }
        k2 += 64;
      }
      if (lane == 0) after_s[x] = below(h, k2) - below(h, k + 1);
    }
    __syncthreads();
    // Entries of loaded block x at or below v (strict: below v), without those
    // before the head's start, and with the still blocks that follow.
    auto entries = [&](int x, double v, bool strict) -> int {
      const double* p = blk + x * kBlk;
      int a = 0, e = kBlk;
      while (a < e) {
        const int mid = (a + e) >> 1;
        if (strict ? p[mid] >= v : p[mid] > v) e = mid;
        else a = mid + 1;
      }
      const int h = sh_s[x], k = sk_s[x];
      const int skip = k == ks_s[h] ? s_s[h] - k * kBlk : 0;
      const int real = min(kBlk, n - 1 - k * kBlk);  // increments up to n-2
      return max(min(a, real) - skip, 0) + (a >= real ? after_s[x] : 0);
    };
    // Stage C.  T: the smallest entry such that those at or below it reach R.
    int64_t base = 0;
    for (int h = 0; h < H; ++h) base += lt_s[h];
    int GS = 1;
    while (GS < ns) GS *= 2;
    const int NS = kAllocThreads / GS;
    int32_t* pc = &pcount[0][0];
    if (tid < ns) {
      const int h = sh_s[tid], k = sk_s[tid];
      il[0][tid] = k == ks_s[h] ? s_s[h] - k * kBlk : 0;
      ir[0][tid] = min(kBlk, n - 1 - k * kBlk);
    }
    if (tid == 0) {
      best_s[0] = ~0ull;
      fail_s[0] = 0ull;
      open_s[0] = 1;
    }
    __syncthreads();
    const int sv = tid / GS, sx = tid % GS;
    rounds = 0;
    while (open_s[0]) {
      if (++rounds > 64) {
        if (tid == 0) *flag = 0;
        return;
      }
      int cnt = 0;
      for (int x = 0; x < ns; ++x) cnt += ir[0][x] - il[0][x];
      const int stride = (cnt + NS - 1) / NS;
      pc[tid] = 0;
      __syncthreads();
      int idx = sv * stride;
      const bool live = idx < cnt;
      double v = 0.0;
      if (live) {
        int x = 0;
        while (idx >= ir[0][x] - il[0][x]) {
          idx -= ir[0][x] - il[0][x];
          ++x;
        }
        v = blk[x * kBlk + il[0][x] + idx];
        if (sx < ns) atomicAdd(&pc[sv], entries(sx, v, false));
      }
      __syncthreads();
      if (live && sx == 0) {
        if (base + pc[sv] >= R)
          atomicMin((unsigned long long*)&best_s[0], (unsigned long long)dkey(v));
        else
          atomicMax((unsigned long long*)&fail_s[0], (unsigned long long)dkey(v));
      }
      __syncthreads();
      if (tid < ns) {
        const double* p = blk + tid * kBlk;
        auto above = [&](int a, int e, uint64_t key) {
          while (a < e) {
            const int mid = (a + e) >> 1;
            if (dkey(p[mid]) > key) e = mid;
            else a = mid + 1;
          }
          return a;
        };
        int a = il[0][tid], e = ir[0][tid];
        if (fail_s[0] != 0ull) a = above(a, e, fail_s[0]);
        if (best_s[0] != ~0ull) e = above(a, e, best_s[0] - 1);  // not the best's equals
        il[0][tid] = a;
        ir[0][tid] = e;
      }
      __syncthreads();
      if (tid == 0) {
        bool more = false;
        if (stride > 1)
          for (int x = 0; x < ns; ++x)
            if (il[0][x] < ir[0][x]) more = true;
        open_s[0] = more ? 1 : 0;
      }
      __syncthreads();
    }
    // Budgets: everything keyed below T, then the increments keyed T, by head.
    const double T = dval(best_s[0]);
    if (tid < H) le_s[tid] = lt_s[tid];
    __syncthreads();
    if (tid < ns) {
      atomicAdd(&lt_s[sh_s[tid]], entries(tid, T, true));
      atomicAdd(&le_s[sh_s[tid]], entries(tid, T, false));
    }
    __syncthreads();
    if (tid == 0) {
      int64_t rem = R;
      for (int h = 0; h < H; ++h) rem -= lt_s[h];
      for (int h = 0; h < H; ++h) {
        const int64_t eq = le_s[h] - lt_s[h];
        const int64_t take = rem < eq ? rem : eq;
        rem -= take;
        s_s[h] += (int32_t)(lt_s[h] + take);
      }
    }
    __syncthreads();
  }
  if (tid < H) budgets[u0 + tid] = s_s[tid];
  if (tid == 0) {
    *flag = 1;
    if (stats) {
      stats[((int64_t)l * g.B + b) * 3 + 0] = R;
      stats[((int64_t)l * g.B + b) * 3 + 1] = (int64_t)(t_bisect - t_start);
      stats[((int64_t)l * g.B + b) * 3 + 2] = (int64_t)(wall_clock64() - t_bisect);
    }
  }
}

__global__ __launch_bounds__(kAllocThreads) void allocate_kernel(
    Geo g, SeqTab st, const float* __restrict__ curves, const float* __restrict__ cmin,
    const float* __restrict__ cmaxb, const int32_t* __restrict__ cpos,
    const double* __restrict__ dmax, int32_t nblk_max, int32_t steps,
    int32_t* __restrict__ budgets, int64_t* __restrict__ stats, int32_t K, int32_t* sync,
    const int32_t* __restrict__ done) {
  // 64 KB of LDS: the half-block minima during the bisection, the
  // block-level running maxima of the marginals during the repair.
  __shared__ __align__(16) unsigned char pool[kLdsItems * 8];
  float2* mcache = reinterpret_cast<float2*>(pool);  // half-block minima
  double* pbm = reinterpret_cast<double*>(pool);
  __shared__ int32_t cand[kCandCap];
  __shared__ double fbest[64];
  __shared__ int32_t bbest[64], kstar[64];
  __shared__ float cbest[64], cprev[64];  // curve values at bbest and bprev
  __shared__ int32_t bprev[64];           // previous argmin (-1: none)
  // One region for three phases: the smallest position of each block's
  // minimum (bisection), the repair search's cached curve blocks, one per
  // (threshold, head) half-wave, and the sequential repair's curve windows.
  constexpr size_t kAuxA = (size_t)kLdsItems * 4, kAuxB = (size_t)kHeadGroup * kRcStride * 4,
                   kAuxC = (size_t)64 * (kRepairWin + 1) * 4;
  constexpr size_t kAux = kAuxA > kAuxB ? (kAuxA > kAuxC ? kAuxA : kAuxC) : (kAuxB > kAuxC ? kAuxB : kAuxC);
  __shared__ __align__(16) unsigned char aux[kAux];
  int32_t* mpos = reinterpret_cast<int32_t*>(aux);
  float* rcache = reinterpret_cast<float*>(aux);
  float(*win)[kRepairWin + 1] = reinterpret_cast<float(*)[kRepairWin + 1]>(aux);
  __shared__ int32_t rkey[kHeadGroup];
  __shared__ int32_t sfirst;  // (head << 16) | block of each cached block (-1: none)
  __shared__ float cres_c[kCandCap];
  __shared__ int32_t bcur[64], bhi[64];
  __shared__ double redf[kAllocWaves];
  __shared__ double cres_f[kCandCap];
  __shared__ int32_t cres_b[kCandCap];
  __shared__ int32_t ncand, scan_pos;
  __shared__ int64_t cnt_lt[64], cnt_le[64];
  __shared__ int64_t cnt_j[64];  // per (threshold, head) counts of the repair search
  __shared__ double tlam[kTreeMax], tlo[kTreeMax], thi[kTreeMax];  // node multipliers
  __shared__ int64_t tsum[kTreeMax];                                // node budget sums
  __shared__ int32_t ticket;

  // With K > 1 workgroups per (layer, sequence), groups are formed from an
  // atomic ticket in arrival order: a workgroup waits only for the others of
  // its group, and the lowest unfinished group either has every member
  // started or holds every started workgroup, so groups always complete.
  int bl, l, node = 0, grp = 0;
  if (K > 1) {
    if (threadIdx.x == 0) ticket = atomicAdd(&sync[0], 1);
    __syncthreads();
    grp = ticket / K;
    node = ticket - grp * K;
    bl = grp % st.count;
    l = grp / st.count;
  } else {
    bl = blockIdx.x;
    l = blockIdx.y;
  }
  if (bl >= st.count || l >= g.L) return;
  const int b = st.first + bl;
  if (done && done[(int64_t)l * g.B + b]) return;  // a whole group returns together
  const int n = st.len[bl];
  const int64_t tok0 = st.start[bl];
  const int64_t B_real = st.b_real[bl];
  const int bmin = st.b_min[bl];
  const int H = g.H;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int sub = tid & 31;
  const int hg = tid >> 5;
  const int nblk = (n + kBlk - 1) / kBlk;
  const int kfirst = bmin / kBlk;
  const bool fast = H * nblk <= kLdsItems;
  const uint64_t t_start = wall_clock64();

  // lambda_hi = 2 max c + 1 over every head and b in [0, n-1]
  double cm = 0.0;
  for (int i = tid; i < H * nblk; i += kAllocThreads) {
    const int h = i / nblk, k = i % nblk;
    cm = fmax(cm, (double)cmaxb[unit_index(g, l, b, h) * nblk_max + k]);
  }
  cm = wave_max(cm);
  if (lane == 0) redf[wave] = cm;
  if (fast) {
    for (int i = tid; i < H * nblk; i += kAllocThreads) {
      const int h = i / nblk, k = i % nblk;
      mcache[i] = reinterpret_cast<const float2*>(cmin)[unit_index(g, l, b, h) * nblk_max + k];
      mpos[i] = cpos[unit_index(g, l, b, h) * nblk_max + k];
    }
  }
  if (tid < 64) bprev[tid] = -1;
  __syncthreads();
  for (int w = 0; w < kAllocWaves; ++w) cm = fmax(cm, redf[w]);
  double lo = 0.0, hi = 2.0 * cm + 1.0;

  // minimum of c over block k of head h
  auto mh_at = [&](int h, int k) -> float {
    const float2 m = fast ? mcache[h * nblk + k]
                          : reinterpret_cast<const float2*>(cmin)[unit_index(g, l, b, h) * nblk_max + k];
    return fminf(m.x, m.y);
  };
  // Whether block k of head h (LDS item i) may hold a point undercutting the
  // head's best (f*, b*): per half, every point b of it has (f(b), b) >=
  // (fma(lam, b0, min c), b0) lexicographically.
  auto undercuts = [&](int i, int h, int k, double lam) -> bool {
    const float2 m = mcache[i];
    const int b0a = max(k * kBlk, bmin), b0b = max(k * kBlk + kBlk / 2, bmin);
    const bool a = k * kBlk + kBlk / 2 - 1 >= bmin &&
                   lex_less(fma(lam, (double)b0a, (double)m.x), b0a, fbest[h], bbest[h]);
    return a || lex_less(fma(lam, (double)b0b, (double)m.y), b0b, fbest[h], bbest[h]);
  };

  // Per head, the block with the smallest bound fma(lambda, b0, min c) is
  // evaluated exactly by 32 threads: (fbest, bbest) is then an exact upper
  // bound of the head's minimum and kstar its block.
  auto best_bound = [&](double lam) {
    for (int h0 = 0; h0 < H; h0 += kHeadGroup) {
      const int h = h0 + hg;
      if (h < H) {
        const float* ch = curves + lht_base(g, l, h, tok0);
        double lbest = INFINITY;
        int kb_ = 0x7fffffff;
        for (int k = kfirst + sub; k < nblk; k += 32) {
          const int b0 = max(k * kBlk, bmin);
          const double lb = fma(lam, (double)b0, (double)mh_at(h, k));
          if (lex_less(lb, k, lbest, kb_)) {
            lbest = lb;
            kb_ = k;
          }
        }
        const int ks = half_wave_min(lbest, kb_).b;
        double f = INFINITY;
        int bb = 0x7fffffff;
        const int lo_b = max(ks * kBlk, bmin), hi_b = min(ks * kBlk + kBlk - 1, n - 1);
        float cv[kBlk / 32];
#pragma unroll
        for (int i = 0; i < kBlk / 32; ++i) {
          const int x = ks * kBlk + sub + 32 * i;
          cv[i] = (x >= lo_b && x <= hi_b) ? ch[x] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < kBlk / 32; ++i) {
          const int x = ks * kBlk + sub + 32 * i;
          if (x >= lo_b && x <= hi_b) {
            const double v = fma(lam, (double)x, (double)cv[i]);
            if (lex_less(v, x, f, bb)) {
              f = v;
              bb = x;
            }
          }
        }
        const BestFB r = half_wave_min(f, bb);
        if (sub == 0) {
          fbest[h] = r.f;
          bbest[h] = r.b;
          kstar[h] = ks;
        }
      }
    }
    __syncthreads();
  };

  // argmin over [bmin, n-1] of fma(lam, b, c_h(b)) for every head -> out[h],
  // for problems whose block minima do not fit in LDS: per-head pruned scans
  auto evaluate_scan = [&](double lam, int32_t* out) {
    best_bound(lam);
    {
      // every other block re-checked by its head's 32 threads
      for (int h0 = 0; h0 < H; h0 += kHeadGroup) {
        const int h = h0 + hg;
        if (h < H) {
          const float* ch = curves + lht_base(g, l, h, tok0);
          double f = fbest[h];
          int bb = bbest[h];
          for (int k = kfirst + sub; k < nblk; k += 32) {
            if (k == kstar[h]) continue;
            const int b0 = max(k * kBlk, bmin);
            const double lb = fma(lam, (double)b0, (double)mh_at(h, k));
            if (!lex_less(lb, b0, f, bb)) continue;
            const int hi_b = min(k * kBlk + kBlk - 1, n - 1);
            for (int x = b0; x <= hi_b; ++x) {
              const double v = fma(lam, (double)x, (double)ch[x]);
              if (lex_less(v, x, f, bb)) {
                f = v;
                bb = x;
              }
            }
          }
          const BestFB r = half_wave_min(f, bb);
          if (sub == 0) {
            fbest[h] = r.f;
            bbest[h] = r.b;
          }
        }
      }
      __syncthreads();
    }
    if (tid < H) out[tid] = bbest[tid];
    __syncthreads();
  };

  // The same argmin with the block minima in LDS, in rounds of at most
  // kCandCap candidate blocks (used when one round cannot hold them all).
  //  1. per head, the block with the smallest bound is evaluated exactly
  //     (32 threads per head): an exact upper bound (f*, b*) of the minimum;
  //  2. every other block whose bound undercuts (f*, b*) is a candidate;
  //     candidates of all heads are gathered (up to kCandCap per round) and
  //     evaluated one block per wave, all loads of a round in flight at once;
  //  3. per head, the smallest (f, b) over its candidates and (f*, b*).
  // Blocks left out cannot hold the answer (ties favour smaller b), so the
  // result is the full scan's.
  auto evaluate_rounds = [&](double lam, int32_t* out) {
    best_bound(lam);
    if (tid == 0) scan_pos = 0;
    __syncthreads();
    const int nitems = H * nblk;
    while (true) {
      // gather candidates from scan_pos on, until the list is full
      if (tid == 0) ncand = 0;
      __syncthreads();
      const int start = scan_pos;
      int stop = nitems;
      for (int i0 = start; i0 < nitems; i0 += kAllocThreads) {
        const int i = i0 + tid;
        bool take = false;
        int h = 0, k = 0;
        if (i < nitems) {
          h = i / nblk;
          k = i - h * nblk;
          if (k >= kfirst && k != kstar[h]) take = undercuts(i, h, k, lam);
        }
        const uint64_t m = __ballot(take);
        int slot0 = 0;
        if (lane == 0 && m) slot0 = atomicAdd(&ncand, __popcll(m));
        slot0 = __builtin_amdgcn_readfirstlane(slot0);
        const int slot = slot0 + (int)count_below64(m);
        if (take && slot < kCandCap) cand[slot] = (h << 16) | k;
        __syncthreads();
        if (ncand > kCandCap) {  // overflow: this sweep is scanned again next round
          stop = i0;
          break;
        }
        if (ncand == kCandCap) {  // full: resume after this sweep
          stop = i0 + kAllocThreads;
          break;
        }
      }
      __syncthreads();
      const int C = min(ncand, kCandCap);
      // evaluate: one candidate block per wave, up to 4 per wave per batch
      for (int c0 = wave; c0 < C; c0 += 4 * kAllocWaves) {
        float cv[4][kBlk / 64];
        int it[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = c0 + q * kAllocWaves;
          it[q] = c < C ? cand[c] : -1;
          const int hq = it[q] < 0 ? 0 : (it[q] >> 16), kq = it[q] < 0 ? 0 : (it[q] & 0xffff);
          const float* ch = curves + lht_base(g, l, hq, tok0);
#pragma unroll
          for (int e = 0; e < kBlk / 64; ++e) {
            const int x = kq * kBlk + lane + 64 * e;
            cv[q][e] = (it[q] >= 0 && x >= bmin && x <= n - 1) ? ch[x] : 0.f;
          }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (it[q] < 0) continue;
          const int kq = it[q] & 0xffff;
          double f = INFINITY;
          int bb = 0x7fffffff;
#pragma unroll
          for (int e = 0; e < kBlk / 64; ++e) {
            const int x = kq * kBlk + lane + 64 * e;
            if (x >= bmin && x <= n - 1) {
              const double v = fma(lam, (double)x, (double)cv[q][e]);
              if (lex_less(v, x, f, bb)) {
                f = v;
                bb = x;
              }
            }
          }
          const BestFB r = wave_lexmin(f, bb);
          if (lane == 0) {
            cres_f[c0 + q * kAllocWaves] = r.f;
            cres_b[c0 + q * kAllocWaves] = r.b;
          }
        }
      }
      __syncthreads();
      // per head: fold the candidates' minima into (f*, b*), 32 threads a head
      for (int h0 = 0; h0 < H; h0 += kHeadGroup) {
        const int h = h0 + hg;
        if (h < H) {
          double f = INFINITY;
          int bb = 0x7fffffff;
          for (int c = sub; c < C; c += 32) {
            if ((cand[c] >> 16) == h && lex_less(cres_f[c], cres_b[c], f, bb)) {
              f = cres_f[c];
              bb = cres_b[c];
            }
          }
          const BestFB r = half_wave_min(f, bb);
          if (sub == 0 && lex_less(r.f, r.b, fbest[h], bbest[h])) {
            fbest[h] = r.f;
            bbest[h] = r.b;
          }
        }
      }
      if (tid == 0) scan_pos = stop;
      __syncthreads();
      if (stop >= nitems) break;
    }
    if (tid < H) {
      out[tid] = bbest[tid];
      bprev[tid] = -1;
    }
    __syncthreads();
  };

  // The argmin with an upper bound that needs no global load: per head the
  // best of (a) the first position of each block's minimum, for blocks whose
  // minimum lies at or after b_min (an actual point of the curve, its value
  // in LDS), and (b) the previous argmin with its curve value.  Every block
  // whose bound undercuts it is a candidate, gathered in one sweep and
  // evaluated one block per wave; if more than kCandCap qualify, the rounds
  // above take over.  As there, blocks left out cannot hold the answer.
  auto evaluate_fast = [&](double lam, int32_t* out) {
    for (int h0 = 0; h0 < H; h0 += kHeadGroup) {
      const int h = h0 + hg;
      if (h < H) {
        double f = INFINITY;
        int bb = 0x7fffffff;
        float cb = 0.f;
#pragma unroll 4
        for (int k = kfirst + sub; k < nblk; k += 32) {
          const int p = mpos[h * nblk + k];
          if (p >= bmin) {
            const float cv = fminf(mcache[h * nblk + k].x, mcache[h * nblk + k].y);
            const double v = fma(lam, (double)p, (double)cv);
            if (lex_less(v, p, f, bb)) {
              f = v;
              bb = p;
              cb = cv;
            }
          }
        }
        if (sub == 0 && bprev[h] >= 0) {
          const double v = fma(lam, (double)bprev[h], (double)cprev[h]);
          if (lex_less(v, bprev[h], f, bb)) {
            f = v;
            bb = bprev[h];
            cb = cprev[h];
          }
        }
        lexmin_fbc<32>(f, bb, cb);
        if (sub == 0) {
          fbest[h] = f;
          bbest[h] = bb;
          cbest[h] = cb;
        }
      }
    }
    if (tid == 0) ncand = 0;
    __syncthreads();
    const int nitems = H * nblk;
    for (int i0 = 0; i0 < nitems; i0 += kAllocThreads) {
      const int i = i0 + tid;
      bool take = false;
      int h = 0, k = 0;
      if (i < nitems) {
        h = i / nblk;
        k = i - h * nblk;
        if (k >= kfirst) take = undercuts(i, h, k, lam);
      }
      const uint64_t m = __ballot(take);
      int slot0 = 0;
      if (lane == 0 && m) slot0 = atomicAdd(&ncand, __popcll(m));
      slot0 = __builtin_amdgcn_readfirstlane(slot0);
      const int slot = slot0 + (int)count_below64(m);
      if (take && slot < kCandCap) cand[slot] = (h << 16) | k;
    }
    __syncthreads();
    const int C = ncand;
    if (C > kCandCap) {
      evaluate_rounds(lam, out);
      return;
    }
    // evaluate: each wave takes a run of `per` consecutive candidates (up to
    // 9, the most whose loads fit in flight in the registers), the
    // candidates spread evenly over the waves; the sweep lists them in (head, block) order, so a run
    // mostly belongs to one head: lanes keep a running best over the run's
    // positions and the wave reduces once per head change, recording the
    // result at that head's last candidate of the run (the others get +inf)
    constexpr int QB = 9;
    const int per = min(QB, (C + kAllocWaves - 1) / kAllocWaves);
    for (int c0 = wave * per; c0 < C; c0 += per * kAllocWaves) {
      float cv[QB][kBlk / 64];
      int it[QB];
#pragma unroll
      for (int q = 0; q < QB; ++q) {
        const int c = c0 + q;
        it[q] = (q < per && c < C) ? cand[c] : -1;
        const int hq = it[q] < 0 ? 0 : (it[q] >> 16), kq = it[q] < 0 ? 0 : (it[q] & 0xffff);
        const float* ch = curves + lht_base(g, l, hq, tok0);
#pragma unroll
        for (int e = 0; e < kBlk / 64; ++e) {
          const int x = kq * kBlk + lane + 64 * e;
          cv[q][e] = (it[q] >= 0 && x >= bmin && x <= n - 1) ? ch[x] : 0.f;
        }
      }
      double f = INFINITY;
      int bb = 0x7fffffff;
      float cb = 0.f;
#pragma unroll
      for (int q = 0; q < QB; ++q) {
        if (it[q] < 0) break;
        const int kq = it[q] & 0xffff;
#pragma unroll
        for (int e = 0; e < kBlk / 64; ++e) {
          const int x = kq * kBlk + lane + 64 * e;
          if (x >= bmin && x <= n - 1) {
            const double v = fma(lam, (double)x, (double)cv[q][e]);
            if (lex_less(v, x, f, bb)) {
              f = v;
              bb = x;
              cb = cv[q][e];
            }
          }
        }
        const bool last = q + 1 == QB || it[q + 1] < 0 || (it[q + 1] >> 16) != (it[q] >> 16);
        if (last) {
          lexmin_fbc<64>(f, bb, cb);
          if (lane == 0) {
            cres_f[c0 + q] = f;
            cres_b[c0 + q] = bb;
            cres_c[c0 + q] = cb;
          }
          f = INFINITY;
          bb = 0x7fffffff;
          cb = 0.f;
        } else if (lane == 0) {
          cres_f[c0 + q] = INFINITY;
          cres_b[c0 + q] = 0x7fffffff;
        }
      }
    }
    __syncthreads();
    // per head: fold the candidates' minima into (f*, b*), 32 threads a head
    for (int h0 = 0; h0 < H; h0 += kHeadGroup) {
      const int h = h0 + hg;
      if (h < H) {
        double f = fbest[h];
        int bb = bbest[h];
        float cb = cbest[h];
        for (int c = sub; c < C; c += 32) {
          if ((cand[c] >> 16) == h && lex_less(cres_f[c], cres_b[c], f, bb)) {
            f = cres_f[c];
            bb = cres_b[c];
            cb = cres_c[c];
          }
        }
        lexmin_fbc<32>(f, bb, cb);
        if (sub == 0) {
          out[h] = bb;
          bprev[h] = bb;
          cprev[h] = cb;
        }
      }
    }
    __syncthreads();
  };
  auto evaluate = [&](double lam, int32_t* out) {
    if (fast)
      evaluate_fast(lam, out);
    else
      evaluate_scan(lam, out);
  };

  // Bisection on lambda: lambda = (lo + hi) / 2, then lo = lambda if the
  // budgets at lambda sum above B_real, else hi = lambda (and bhi = the
  // budgets there).
  // The budgets at the initial lambda_hi are needed only when no step lowers
  // it; they are then evaluated after the steps.
  bool have_bhi = false;
  if (K <= 1) {
    for (int t = 0; t < steps; ++t) {
      const double lam = (lo + hi) / 2.0;
      evaluate(lam, bcur);
      int64_t sum = 0;
      for (int h = 0; h < H; ++h) sum += bcur[h];
      if (sum > B_real) {
        lo = lam;
      } else {
        hi = lam;
        have_bhi = true;
        if (tid < H) bhi[tid] = bcur[tid];
      }
      __syncthreads();
    }
    if (!have_bhi) evaluate(hi, bhi);
  } else {
    // The same steps, lev at a time: the multipliers of the next lev steps
    // form a binary tree (node i's children 2i+1 after hi = lambda_i and
    // 2i+2 after lo = lambda_i), each computed from its interval exactly as
    // the step-by-step bisection would.  The group's workgroup `node`
    // evaluates node `node`, the sums are exchanged through global memory,
    // and every workgroup then follows the same path down the tree.  Only
    // node 0 keeps bhi and goes on to the repair.
    const int lev_max = 31 - __clz(K + 1);
    int64_t* xsum = reinterpret_cast<int64_t*>(sync + kSyncSum) + (size_t)grp * 2 * kTreeMax;
    int32_t* xarg = sync + kSyncArg + (size_t)grp * 2 * kTreeMax * 64;
    int t = 0, pass = 0;
    // node 0: the argmins of the last node whose sum lowered lambda_hi, kept
    // in flight in registers while the next pass evaluates (the release of
    // the next publication waits for them) and stored once after the loop
    int32_t arg_hi = 0;
    while (t < steps) {
      const int lv = min(lev_max, steps - t);
      const int nl = (1 << lv) - 1;
      const int par = pass & 1;
      if (tid == 0) {
        tlo[0] = lo;
        thi[0] = hi;
        for (int i = 0; i < nl; ++i) {
          tlam[i] = (tlo[i] + thi[i]) / 2.0;
          if (2 * i + 2 < nl) {
            tlo[2 * i + 1] = tlo[i];
            thi[2 * i + 1] = tlam[i];
            tlo[2 * i + 2] = tlam[i];
            thi[2 * i + 2] = thi[i];
          }
        }
      }
      __syncthreads();
      if (node < nl) {
        evaluate(tlam[node], bcur);
        if (tid < H)
          __hip_atomic_store(&xarg[(par * kTreeMax + node) * 64 + tid], bcur[tid],
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      // Exchange.  Each evaluating node publishes its budget sum tagged with
      // the pass, released after its argmins (ordered before it by the
      // barrier); lanes 0..nl-1 of wave 0 poll one node's slot each with
      // coherent (agent-scope atomic) loads until every tag shows this pass,
      // and so hold the sums when the wait ends.  No acquire fence is needed
      // (the argmins are read with the same loads; an agent-scope acquire
      // would also invalidate the compute die's L2, which holds the curve
      // blocks the next evaluation rereads).  Slots alternate by pass parity:
      // a node publishes pass p + 2 only after it has seen every node's pass
      // p + 1, which each node publishes after reading pass p.
      __syncthreads();
      if (node < nl && tid == 0) {
        int64_t sum = 0;
        for (int h = 0; h < H; ++h) sum += bcur[h];
        __hip_atomic_store(&xsum[par * kTreeMax + node], ((int64_t)(pass + 1) << 48) | sum,
                           __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (wave == 0) {
        int64_t v = 0;
        int spins = 0;
        while (true) {
          if (lane < nl)
            v = __hip_atomic_load(&xsum[par * kTreeMax + lane], __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
          if (__ballot(lane < nl && (v >> 48) != (int64_t)(pass + 1)) == 0) break;
          __builtin_amdgcn_s_sleep(1);
          if (++spins > (1 << 22)) {  // a member never published: give up, report
            if (lane == 0 && g.status) *g.status = CERTKV_EHIP;
            break;
          }
        }
        if (lane < nl) tsum[lane] = v & (((int64_t)1 << 48) - 1);
      }
      __syncthreads();
      int nd = 0, last = -1;
      for (int j = 0; j < lv; ++j) {
        if (tsum[nd] > B_real) {
          lo = tlam[nd];
          nd = 2 * nd + 2;
        } else {
          hi = tlam[nd];
          last = nd;
          nd = 2 * nd + 1;
        }
      }
      if (node == 0 && last >= 0 && tid < H)
        arg_hi = __hip_atomic_load(&xarg[(par * kTreeMax + last) * 64 + tid], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
      have_bhi = have_bhi || last >= 0;
      __syncthreads();  // every thread has walked the tree before tid 0 rebuilds it
      t += lv;
      ++pass;
    }
    if (node != 0) return;
    if (have_bhi && tid < H) bhi[tid] = arg_hi;
    __syncthreads();
    if (!have_bhi) evaluate(hi, bhi);
  }
  const uint64_t t_bisect = wall_clock64();
  // A head whose curve holds no comparable value from b_min on (all NaN) has
  // no argmin: it starts the repair from b_min.
  if (tid < H && (bhi[tid] < bmin || bhi[tid] > n - 1)) bhi[tid] = bmin;
  __syncthreads();

  int64_t sum0 = 0;
  for (int h = 0; h < H; ++h) sum0 += bhi[h];
  const int64_t R = B_real - sum0;
  const int64_t nrep = R >= 0 ? R : -R;
  const int kmax = (n - 2) / kBlk;  // last block holding an increment i <= n-2

  // Number of increments of head h whose key P is < p (le = false) or <= p
  // (le = true); computed by the 32 threads of half-wave `slot` (< kHeadGroup),
  // which keeps the last curve block it scanned in LDS: once the search has
  // narrowed, successive thresholds cross in the same block and the count
  // reads no global memory.
  auto count_head = [&](int h, double p, bool le, int slot) -> int64_t {
    const int s = bhi[h];
    if (s > n - 2) return 0;
    const int ks = s / kBlk;
    auto crosses = [&](double v) { return le ? (v > p) : (v >= p); };
    const double* ph = pbm + h * nblk;
    int lo_k;  // first block whose running max crosses p
    const int key = rkey[slot];
    const int kc = (key >> 16) == h ? (key & 0xffff) : -1;
    if (kc >= ks && kc <= kmax && crosses(ph[kc]) && (kc == ks || !crosses(ph[kc - 1]))) {
      lo_k = kc;
    } else {
      lo_k = ks;
      int hi_k = kmax + 1;
      while (lo_k < hi_k) {
        const int mid = (lo_k + hi_k) >> 1;
        if (crosses(ph[mid])) hi_k = mid;
        else lo_k = mid + 1;
      }
    }
    if (lo_k > kmax) return (int64_t)(n - 1 - s);
    float* rc = rcache + slot * kRcStride;  // c(lo_k kBlk + i), i = 0..kBlk
    if (lo_k != kc) {
      const float* ch = curves + lht_base(g, l, h, tok0);
      float v[(kBlk + 32) / 32];
#pragma unroll
      for (int m = 0; m < (kBlk + 32) / 32; ++m) {
        const int i = sub + 32 * m;
        v[m] = i <= kBlk ? cval(ch[min(lo_k * kBlk + i, n - 1)]) : 0.f;
      }
#pragma unroll
      for (int m = 0; m < (kBlk + 32) / 32; ++m) {
        const int i = sub + 32 * m;
        if (i <= kBlk) rc[i] = v[m];
      }
      // every thread of the half-wave has read rkey above; the block is read
      // back by other threads of the same wave
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (sub == 0) rkey[slot] = (h << 16) | lo_k;
    }
    const int i0 = max(lo_k * kBlk, s), i1 = min(lo_k * kBlk + kBlk - 1, n - 2);
    int first = 0x7fffffff;
#pragma unroll
    for (int m = kBlk / 32 - 1; m >= 0; --m) {
      const int r = sub + 32 * m, i = lo_k * kBlk + r;
      const double d = (double)rc[r + 1] - (double)rc[r];
      if (i >= i0 && i <= i1 && crosses(d)) first = i;
    }
    first = half_min_i32(first);
    return (int64_t)(first - s);
  };
  auto total_count = [&](double p, bool le, int64_t* per_head) -> int64_t {
    for (int h0 = 0; h0 < H; h0 += kHeadGroup) {
      const int h = h0 + hg;
      if (h < H) {
        const int64_t c = count_head(h, p, le, hg);
        if (sub == 0) per_head[h] = c;
      }
    }
    __syncthreads();
    int64_t tot = 0;
    for (int h = 0; h < H; ++h) tot += per_head[h];
    __syncthreads();
    return tot;
  };

  if (R > 0 && fast) {
    // pbm[h*nblk + k] = running max of d_h over [s_h, end of block k] for the
    // blocks k >= block of s_h (s_h = bhi[h]); -inf before it.  The block
    // maxima come into LDS with all threads; each head's running maximum is
    // then a prefix maximum over its blocks by one half-wave (a run of
    // blocks per thread, then a scan of the runs).
    for (int i = tid; i < H * nblk; i += kAllocThreads) {
      const int h = i / nblk, k = i - h * nblk;
      pbm[i] = dmax[unit_index(g, l, b, h) * nblk_max + k];
    }
    if (tid < kHeadGroup) rkey[tid] = -1;
    __syncthreads();
    for (int h0 = 0; h0 < H; h0 += kHeadGroup) {
      const int h = h0 + hg;
      if (h < H) {
        const float* ch = curves + lht_base(g, l, h, tok0);
        const int s = bhi[h];
        const int ks = s / kBlk;
        double dm = -INFINITY;
        if (s <= n - 2) {
          const int e1 = min(ks * kBlk + kBlk - 1, n - 2);
          for (int i = s + sub; i <= e1; i += 32)
            dm = fmax(dm, (double)cval(ch[i + 1]) - (double)cval(ch[i]));
        }
#pragma unroll
        for (int m = 16; m >= 1; m >>= 1) dm = fmax(dm, __shfl_xor(dm, m, 64));
        // block values: the partial first block, then the block maxima up to
        // the last block holding an increment; -inf elsewhere
        double* ph = pbm + h * nblk;
        const bool none = s > n - 2;
        auto val = [&](int k) -> double {
          if (none || k < ks) return -INFINITY;
          if (k == ks) return dm;
          return k <= kmax ? ph[k] : -INFINITY;
        };
        const int per = (nblk + 31) / 32;
        const int k0 = sub * per, k1 = min(nblk, k0 + per);
        double run = -INFINITY;
        for (int k = k0; k < k1; ++k) run = fmax(run, val(k));
        // exclusive prefix maximum of the runs over the half-wave
        double incl = run;
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) {
          const double y = __shfl_up(incl, off, 32);
          if (sub >= off) incl = fmax(incl, y);
        }
        double acc = __shfl_up(incl, 1, 32);
        if (sub == 0) acc = -INFINITY;
        // each thread reads and rewrites only its own blocks, each block's
        // value read just before it is overwritten
        for (int k = k0; k < k1; ++k) {
          acc = fmax(acc, val(k));
          ph[k] = (none || k < ks) ? -INFINITY : acc;
        }
      }
    }
    __syncthreads();
    // smallest key x in [-inf, +inf] with count(P <= x) >= R, by a (J+1)-ary
    // search over the ordered bit patterns (count(P <= +inf) covers every
    // increment): each step counts at J interior points of [klo, khi) at once,
    // one half-wave per (point, head).
    uint64_t klo = dkey(-INFINITY), khi = dkey(INFINITY);
    // A = 2^la <= kHeadGroup / H (at least 2) parts per step, so that the
    // points need no division; (point, head) pairs beyond the half-waves
    // (more than 32 heads) are taken in further rounds
    int la = 1;
    while ((2 << la) <= kHeadGroup / H) ++la;
    const int J = (1 << la) - 1;
    // interior point j: klo + floor(span (j+1) / 2^la), < khi, without overflow
    auto point = [&](uint64_t lo_k, uint64_t span, int j) -> uint64_t {
      return lo_k + (span >> la) * (uint64_t)(j + 1) +
             (((span & (uint64_t)J) * (uint64_t)(j + 1)) >> la);
    };
    while (klo < khi) {
      const uint64_t span = khi - klo;
      for (int gi = hg; gi < J * H; gi += kHeadGroup) {
        const int j = gi / H, h = gi - j * H;
        const int64_t c = count_head(h, dval(point(klo, span, j)), true, hg);
        if (sub == 0) cnt_j[gi] = c;
      }
      __syncthreads();
      // first point whose count reaches R (the counts grow with the point):
      // lane j of wave 0 totals point j over the heads
      if (wave == 0) {
        int64_t c = 0;
        if (lane < J)
          for (int h = 0; h < H; ++h) c += cnt_j[lane * H + h];
        const uint64_t reach = __ballot(lane < J && c >= R);
        if (lane == 0) sfirst = reach ? (int)__builtin_ctzll(reach) : J;
      }
      __syncthreads();
      const int first = sfirst;
      if (first < J) {
        const uint64_t nlo = first > 0 ? point(klo, span, first - 1) + 1 : klo;
        khi = point(klo, span, first);
        klo = nlo;
      } else {
        klo = point(klo, span, J - 1) + 1;
      }
    }
    const double pstar = dval(klo);
    total_count(pstar, false, cnt_lt);
    total_count(pstar, true, cnt_le);
    if (tid == 0) {
      int64_t rem = R;
      for (int h = 0; h < H; ++h) rem -= cnt_lt[h];
      for (int h = 0; h < H; ++h) {
        const int64_t eq = cnt_le[h] - cnt_lt[h];
        const int64_t take = rem < eq ? rem : eq;
        rem -= take;
        bhi[h] = bhi[h] + (int32_t)(cnt_lt[h] + take);
      }
    }
    __syncthreads();
    if (tid < H) budgets[unit_index(g, l, b, tid)] = bhi[tid];
  } else if (tid < 64) {
    // Sequential repair (large problems, or the unreachable removal case).
    const bool act = lane < H;
    int bh = act ? bhi[lane] : 0;
    const float* ch = act ? curves + lht_base(g, l, lane, tok0) : curves;
    int64_t sum = sum0;
    int wbase = bh;  // win[lane][i] = c(wbase + i)
    if (act)
      for (int i = 0; i <= kRepairWin && wbase + i < n; ++i) win[lane][i] = cval(ch[wbase + i]);
    while (sum < B_real) {
      double d = INFINITY;
      if (act && bh < n - 1) {
        if (bh + 1 - wbase > kRepairWin) {
          wbase = bh;
          for (int i = 0; i <= kRepairWin && wbase + i < n; ++i) win[lane][i] = cval(ch[wbase + i]);
        }
        d = (double)win[lane][bh + 1 - wbase] - (double)win[lane][bh - wbase];
      }
      const BestFB r = wave_lexmin(d, act ? lane : 0x7fffffff);
      if (r.f == INFINITY) break;  // unreachable: B_real <= H (n - 1)
      if (lane == r.b) ++bh;
      ++sum;
    }
    while (sum > B_real) {
      double d = INFINITY;
      if (act && bh > bmin) d = (double)cval(ch[bh - 1]) - (double)cval(ch[bh]);
      const BestFB r = wave_lexmin(d, act ? lane : 0x7fffffff);
      if (r.f == INFINITY) break;  // unreachable: H b_min <= B_real
      if (lane == r.b) --bh;
      --sum;
    }
    if (act) budgets[unit_index(g, l, b, lane)] = bh;
  }
  if (stats && tid == 0) {
    stats[((int64_t)l * g.B + b) * 3 + 0] = nrep;
    stats[((int64_t)l * g.B + b) * 3 + 1] = (int64_t)(t_bisect - t_start);
    stats[((int64_t)l * g.B + b) * 3 + 2] = (int64_t)(wall_clock64() - t_bisect);
  }
}

certkv_status run_allocate(const AllocArgs& a, const SeqTab& st, hipStream_t s) {
  // Workgroups per (layer, sequence): a node tree of 3 or 7 when every group
  // of the launch then still has a compute unit per workgroup (one
  // allocation workgroup fills a compute unit's LDS), else 1.
  const int groups = st.count * a.g.L;
  int K = 1;
  if (a.sync && a.steps > 1 && groups <= kSyncGroups) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return CERTKV_EHIP;
    const int cus = device_cus(dev);
    K = 7 * groups <= cus ? 7 : 3 * groups <= cus ? 3 : 1;
  }
  int32_t* sync = K > 1 ? a.sync : nullptr;
  // Tail masses are convex without noise, all of them hull points: no filter.
  const bool hull = a.hull_pts && a.g.stat != 2 && a.g.H * a.nblk_max <= kLdsItems;
  const int nb = hull ? a.chunk_blocks : 8;
  const int nchunk = (a.nblk_max + nb - 1) / nb;
  const dim3 bgrid(a.g.H * st.count * ((nchunk + 3) / 4), a.g.L);
#define CERTKV_BLOCKSTATS(HULL, NB)                                                                \
  CERTKV_LAUNCH("curve_blockstats", (curve_blockstats_kernel<HULL, NB>), bgrid, dim3(256), 0, s,   \
                a.g, st, a.nblk_max, a.curves, a.cmin, a.cmaxb, a.cpos, a.dmax, sync,              \
                (int32_t)kSyncArg, a.hull_pts, a.hull_cnt)
  if (hull) {
    if (nb == 8)
      CERTKV_BLOCKSTATS(true, 8);
    else
      CERTKV_BLOCKSTATS(true, 2);
    CERTKV_LAUNCH("hull_merge", hull_merge_kernel, dim3(a.g.H * st.count, a.g.L),
                  dim3(kMergeThreads), 0, s, a.g, st, a.nblk_max, nb, (const float*)a.cmaxb,
                  a.hull_pts, (const int32_t*)a.hull_cnt, a.unit_cnt, a.unit_max);
    CERTKV_LAUNCH("allocate_hull", allocate_hull_kernel, dim3(st.count, a.g.L), dim3(kAllocThreads),
                  0, s, a.g, st, a.curves, (const double*)a.dmax, a.nblk_max, nb, a.steps,
                  (const uint2*)a.hull_pts, (const int32_t*)a.unit_cnt, (const float*)a.unit_max,
                  a.budgets, a.repairs, a.done);
  } else {
    CERTKV_BLOCKSTATS(false, 8);
  }
#undef CERTKV_BLOCKSTATS
  const int32_t* done = hull ? a.done : nullptr;
  if (K > 1) {
    CERTKV_LAUNCH("allocate", allocate_kernel, dim3((unsigned)(K * groups)), dim3(kAllocThreads), 0,
                  s, a.g, st, a.curves, (const float*)a.cmin, (const float*)a.cmaxb,
                  (const int32_t*)a.cpos, (const double*)a.dmax, a.nblk_max, a.steps, a.budgets,
                  a.repairs, K, a.sync, done);
  } else {
    CERTKV_LAUNCH("allocate", allocate_kernel, dim3(st.count, a.g.L), dim3(kAllocThreads), 0, s,
                  a.g, st, a.curves, (const float*)a.cmin, (const float*)a.cmaxb,
                  (const int32_t*)a.cpos, (const double*)a.dmax, a.nblk_max, a.steps, a.budgets,
                  a.repairs, 1, (int32_t*)nullptr, done);
  }
  return CERTKV_OK;
}

}  // namespace certkv
