// Tail-summary slot and packed-cache compaction.
//
// Per unit the evicted set E is the complement of the kept positions.  The
// slot is the (s)_+-weighted key and value centroid of E; the weights'
// normalizer cancels, so
//   k* = sum_E s_j k_j / sum_E s_j,  v* likewise,  m = sum_E s_j / sum_j s_j.
// When the totals sum_j s_j k_j and sum_j s_j v_j are already known (from the
// scoring and curve kernels) the evicted sums are total minus kept, so only
// the kept rows (about a tenth) are read.  Without the totals, or if the
// evicted mass is below 1/64 of the total (cancellation guard), the evicted
// rows are summed directly instead.
//
// mass      (standalone path only) partial total / evicted score mass;
// gather    (nsplit workgroups per unit) copies a slice of the unit's kept
//           rows into the packed cache and forms fp64 partial weighted sums,
//           of those rows or, for a direct unit, of the evicted rows of a
//           slice of positions;
// finalize  (one workgroup per unit) adds the partials in split order,
//           forms k*, v*, m and appends the slot row.
#include "stages.h"

namespace certkv {

constexpr int kTailThreads = 256;
constexpr int kListTile = 512;  // positions listed at a time by a direct unit's split
constexpr double kComplementMinMass = 1.0 / 64.0;

template <typename T>
__device__ __forceinline__ float elem_f32(const uint4& q, int e);
template <>
__device__ __forceinline__ float elem_f32<uint16_t>(const uint4& q, int e) {
  const uint32_t w = (&q.x)[e >> 1];
  return (e & 1) ? bf16_hi(w) : bf16_lo(w);
}
template <>
__device__ __forceinline__ float elem_f32<float>(const uint4& q, int e) {
  return __uint_as_float((&q.x)[e]);
}

template <typename T>
__device__ __forceinline__ T from_f32(float x);
template <>
__device__ __forceinline__ uint16_t from_f32<uint16_t>(float x) { return f32_to_bf16_rne(x); }
template <>
__device__ __forceinline__ float from_f32<float>(float x) { return x; }

__device__ __forceinline__ bool is_kept(const uint64_t* bmu, int j) {
  return (bmu[j >> 6] >> (j & 63)) & 1ull;
}

// Clear the per-unit kept bitmaps, then set one bit per kept position.
__global__ void bitmap_clear_kernel(uint64_t* __restrict__ bm, int64_t words) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < words) bm[i] = 0ull;
}

// nsplit workgroups share a unit's kept entries: the atomics of one workgroup
// per unit are a serial chain of round trips (two sequences of 65537 and 24001
// keys, 8 heads: 247 us with one).  The bits of one word that neighbouring
// lanes set are joined first: up to 64 atomics to the same word wait for each
// other (a head that keeps almost all of 65537: 30 us, joined 4).
__global__ void bitmap_set_kernel(Geo g, SeqTab st, int32_t nsplit,
                                  const int64_t* __restrict__ kept_offsets,
                                  const int32_t* __restrict__ kept_idx, uint64_t* __restrict__ bm,
                                  int32_t bm_stride) {
  const int split = blockIdx.x % nsplit;
  const int hb = blockIdx.x / nsplit;
  const int h = hb % g.H;
  const int bl = hb / g.H;
  const int l = blockIdx.y;
  if (bl >= st.count) return;
  const int n = st.len[bl];
  const int64_t u = unit_index(g, l, st.first + bl, h);
  const int64_t o0 = kept_offsets[u], o1 = kept_offsets[u + 1];
  const int lane = threadIdx.x & 63;
  for (int64_t i0 = o0 + (int64_t)split * blockDim.x; i0 < o1; i0 += (int64_t)nsplit * blockDim.x) {
    const int64_t i = i0 + threadIdx.x;
    const int j = i < o1 ? kept_idx[i] : -1;
    const bool ok = j >= 0 && j < n;
    const int word = ok ? j >> 6 : -1;
    unsigned long long bits = ok ? 1ull << (j & 63) : 0ull;
    // each lane collects the bits of its word from the lanes that follow it
    // without a break (in any order: joining a later run's bits as well sets
    // no bit that is not to be set); the first lane of a run holds them all
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned long long y = __shfl_down(bits, o, 64);
      const int w = __shfl_down(word, o, 64);
      if (lane + o < 64 && w == word) bits |= y;
    }
    const int before = __shfl_up(word, 1, 64);
    if (ok && (lane == 0 || before != word))
      atomicOr(reinterpret_cast<unsigned long long*>(&bm[u * bm_stride + word]), bits);
  }
}

// Partial total and evicted (s)_+ mass over a slice of positions.
__global__ __launch_bounds__(kTailThreads) void mass_kernel(Geo g, SeqTab st, int32_t nsplit,
                                                            const float* __restrict__ scores,
                                                            const uint64_t* __restrict__ bm,
                                                            int32_t bm_stride,
                                                            double* __restrict__ mpart) {
  __shared__ double red[3][kTailThreads / 64];
  const int split = blockIdx.x % nsplit;
  const int hb = blockIdx.x / nsplit;
  const int h = hb % g.H;
  const int bl = hb / g.H;
  const int l = blockIdx.y;
  if (bl >= st.count) return;
  const int n = st.len[bl];
  const int64_t u = unit_index(g, l, st.first + bl, h);
  const int64_t sbase = lht_base(g, l, h, st.start[bl]);
  const uint64_t* bmu = bm + u * bm_stride;
  const int per = (n + nsplit - 1) / nsplit;
  const int j0 = split * per, j1 = min(n, j0 + per);
  double sa = 0.0, se = 0.0, ne = 0.0;
  for (int j = j0 + threadIdx.x; j < j1; j += kTailThreads) {
    const float s = scores[sbase + j];
    const double sp = s > 0.f ? (double)s : 0.0;
    sa += sp;
    if (!is_kept(bmu, j)) {
      se += sp;
      ne += 1.0;
    }
  }
  sa = wave_sum(sa);
  se = wave_sum(se);
  ne = wave_sum(ne);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    red[0][wave] = sa;
    red[1][wave] = se;
    red[2][wave] = ne;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const int i = threadIdx.x;
    mpart[(u * nsplit + split) * 3 + i] = red[i][0] + red[i][1] + red[i][2] + red[i][3];
  }
}

// A unit's masses and how its evicted sums are formed; the same values in
// the gather (which sums) and in the finalize (which divides).
struct TailMass {
  double all, ev;   // sum of (s)_+ over every key and over the evicted ones
  bool uniform;     // every score zero: uniform weights, masses are counts
  bool direct;      // the evicted rows are summed (else totals minus kept)
};
__device__ __forceinline__ TailMass tail_masses(int64_t u, int n, int nk, int nslice, bool totals,
                                                const double* evicted_sum, const double* total_sum,
                                                const double* mpart) {
  TailMass t;
  double nE;
  if (evicted_sum && total_sum) {
    t.all = total_sum[u];
    t.ev = evicted_sum[u];
    nE = (double)(n - nk);
  } else {
    t.all = t.ev = nE = 0.0;
#pragma unroll 8
    for (int sp = 0; sp < nslice; ++sp) {
      t.all += mpart[(u * nslice + sp) * 3 + 0];
      t.ev += mpart[(u * nslice + sp) * 3 + 1];
      nE += mpart[(u * nslice + sp) * 3 + 2];
    }
  }
  t.uniform = !(t.all > 0.0);
  if (t.uniform) {
    t.all = (double)n;
    t.ev = nE;
  }
  t.direct = t.uniform || !totals || t.ev < kComplementMinMass * t.all;
  return t;
}

// Kept rows of one split: the unit's rows in nsplit parts, none shorter than a
// step of the gather, so that a unit of few rows takes few splits (and its
// finalize reads few partials) while one that keeps almost every row of a
// small launch uses them all.
template <int D, typename T>
struct GatherStep {
  static constexpr int EPL = 16 / sizeof(T);      // elements per 16-byte lane chunk
  static constexpr int LPR = D / EPL;             // lanes per row
  static constexpr int RPS = kTailThreads / LPR;  // rows per load of the workgroup
  static constexpr int UR = 4;                    // loads of a step
  static __device__ __forceinline__ int rows(int nk, int nsplit) {
    return max((nk + nsplit - 1) / nsplit, RPS * UR);
  }
};

// Copy a slice of kept rows to the packed cache and/or accumulate the fp64
// partial weighted key and value sums of the slice.  A direct unit's evicted
// rows are read here, by every split, and not by the unit's one finalize
// workgroup: bound by the row gather (two sequences of 65537 and 24001 keys, 8
// heads, no totals: 84 us for the gather and finalize, 6940 us with the
// sums in the finalize kernel).
template <int D, typename T, bool DO_TAIL, bool DO_COMPACT>
__global__ __launch_bounds__(kTailThreads) void tail_gather_kernel(
    Geo g, SeqTab st, int32_t nsplit, int32_t nslice, bool totals, const uint64_t* __restrict__ bm,
    int32_t bm_stride, const double* __restrict__ mpart, const double* __restrict__ evicted_sum,
    const double* __restrict__ total_sum, const float* __restrict__ scores, const T* __restrict__ kc,
    int64_t k_sl, int64_t k_st, int64_t k_sh, const T* __restrict__ vc, int64_t v_sl,
    int64_t v_st, int64_t v_sh, const int64_t* __restrict__ kept_offsets,
    const int32_t* __restrict__ kept_idx, double* __restrict__ kpart_out,
    T* __restrict__ k_packed, T* __restrict__ v_packed, int32_t* __restrict__ pos_packed) {
  using Step = GatherStep<D, T>;
  constexpr int EPL = Step::EPL, LPR = Step::LPR, RPS = Step::RPS;
  __shared__ double redk[DO_TAIL ? RPS : 1][D];
  __shared__ double redv[DO_TAIL ? RPS : 1][D];
  __shared__ int32_t lpos[DO_TAIL ? kListTile : 1];   // a direct unit's evicted positions
  __shared__ double lwt[DO_TAIL ? kListTile : 1];     // and their weights
  __shared__ int32_t lcnt[DO_TAIL ? kListTile / 64 : 1];

  const int split = blockIdx.x % nsplit;
  const int hb = blockIdx.x / nsplit;
  const int h = hb % g.H;
  const int bl = hb / g.H;
  const int l = blockIdx.y;
  if (bl >= st.count) return;
  const int b = st.first + bl;
  const int n = st.len[bl];
  const int64_t tok0 = st.start[bl];
  const int64_t sbase = lht_base(g, l, h, tok0);
  const int64_t u = unit_index(g, l, b, h);
  const int tid = threadIdx.x;
  const int ri = tid / LPR, ci = tid % LPR;
  const int64_t off = kept_offsets[u];
  const int nk = (int)(kept_offsets[u + 1] - off);
  const int per = Step::rows(nk, nsplit);
  const int i0 = split * per, i1 = min(nk, i0 + per);
  const int64_t poff = off + g.slot * u;  // packed segment start
  const T* kb = kc + (int64_t)l * k_sl + tok0 * k_st + (int64_t)h * k_sh;
  const T* vb = vc + (int64_t)l * v_sl + tok0 * v_st + (int64_t)h * v_sh;

  double ak[EPL], av[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) ak[e] = av[e] = 0.0;
  // Four rows per lane group per step: their indices, then their rows and
  // scores, are loaded together so that each step waits for two round trips.
  constexpr int UR = Step::UR;
  bool direct = false, uniform = false;
  if (DO_TAIL) {
    const TailMass tm = tail_masses(u, n, nk, nslice, totals, evicted_sum, total_sum, mpart);
    direct = tm.direct;
    uniform = tm.uniform;
  }
  if (!direct && i0 >= i1) return;  // (the whole workgroup; the finalize skips its partial)
  if (DO_TAIL && direct) {
    // The evicted positions of this split's slice that carry weight, listed in
    // position order a tile at a time (a ballot per round and wave, then the
    // prefix of the (round, wave) counts), and their rows summed in list order.
    constexpr int LR = kListTile / kTailThreads, LW = kTailThreads / 64;
    const int lane = tid & 63, wave = tid >> 6;
    const uint64_t* bmu = bm + u * bm_stride;
    const int jper = (n + nsplit - 1) / nsplit;
    const int js = min(n, split * jper), je = min(n, js + jper);
    for (int j0 = js; j0 < je; j0 += kListTile) {
      double w[LR];
      uint64_t bal[LR];
#pragma unroll
      for (int r = 0; r < LR; ++r) {
        const int j = j0 + r * kTailThreads + tid;
        const int jc = min(j, n - 1);
        const float s = scores[sbase + jc];
        w[r] = uniform ? 1.0 : (s > 0.f ? (double)s : 0.0);
        const bool take = j < je && w[r] != 0.0 && !is_kept(bmu, jc);
        bal[r] = __ballot(take);
        if (lane == 0) lcnt[r * LW + wave] = (int)__popcll(bal[r]);
      }
      __syncthreads();
      int cnt = 0, start[LR];
#pragma unroll
      for (int r = 0; r < LR; ++r) {
#pragma unroll
        for (int x = 0; x < LW; ++x) {
          if (x == wave) start[r] = cnt;
          cnt += lcnt[r * LW + x];
        }
      }
#pragma unroll
      for (int r = 0; r < LR; ++r) {
        if ((bal[r] >> lane) & 1ull) {
          const int p = start[r] + (int)__builtin_amdgcn_mbcnt_hi(
              (uint32_t)(bal[r] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal[r], 0u));
          lpos[p] = j0 + r * kTailThreads + tid;
          lwt[p] = w[r];
        }
      }
      __syncthreads();
      for (int i = ri; i < cnt; i += RPS * UR) {
        // entries past the list read its last one again, with weight zero
        uint4 kq[UR], vq[UR];
        double ww[UR];
#pragma unroll
        for (int q = 0; q < UR; ++q) {
          const int x = min(i + q * RPS, cnt - 1);
          const int j = lpos[x];
          ww[q] = i + q * RPS < cnt ? lwt[x] : 0.0;
          kq[q] = *reinterpret_cast<const uint4*>(kb + (int64_t)j * k_st + ci * EPL);
          vq[q] = *reinterpret_cast<const uint4*>(vb + (int64_t)j * v_st + ci * EPL);
        }
#pragma unroll
        for (int q = 0; q < UR; ++q) {
          if (i + q * RPS >= cnt) continue;
#pragma unroll
          for (int e = 0; e < EPL; ++e) {
            ak[e] = fma(ww[q], (double)elem_f32<T>(kq[q], e), ak[e]);
            av[e] = fma(ww[q], (double)elem_f32<T>(vq[q], e), av[e]);
          }
        }
      }
      __syncthreads();  // the list is read before the next tile rewrites it
    }
  }
  if (DO_COMPACT || !direct) for (int i = i0 + ri; i < i1; i += RPS * UR) {
    // The entries past the run read a clamped one and fetch its row again,
    // unused: no load sits behind a branch, so none waits for itself.
    int j[UR];
#pragma unroll
    for (int q = 0; q < UR; ++q)
      j[q] = min(max(kept_idx[off + min(i + q * RPS, i1 - 1)], 0), n - 1);  // caller indices clamped
    uint4 kq[UR], vq[UR];
    float sv[UR];
#pragma unroll
    for (int q = 0; q < UR; ++q) {
      kq[q] = *reinterpret_cast<const uint4*>(kb + (int64_t)j[q] * k_st + ci * EPL);
      vq[q] = *reinterpret_cast<const uint4*>(vb + (int64_t)j[q] * v_st + ci * EPL);
      sv[q] = DO_TAIL ? scores[sbase + j[q]] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < UR; ++q) {
      if (i + q * RPS >= i1) continue;
      const int ii = i + q * RPS;
      if (DO_COMPACT) {
        *reinterpret_cast<uint4*>(k_packed + (poff + ii) * D + ci * EPL) = kq[q];
        *reinterpret_cast<uint4*>(v_packed + (poff + ii) * D + ci * EPL) = vq[q];
        if (ci == 0) pos_packed[poff + ii] = j[q];
      }
      if (DO_TAIL && !direct) {
        const double w = sv[q] > 0.f ? (double)sv[q] : 0.0;
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          ak[e] = fma(w, (double)elem_f32<T>(kq[q], e), ak[e]);
          av[e] = fma(w, (double)elem_f32<T>(vq[q], e), av[e]);
        }
      }
    }
  }
  if (DO_TAIL) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      redk[ri][ci * EPL + e] = ak[e];
      redv[ri][ci * EPL + e] = av[e];
    }
    __syncthreads();
    for (int d = tid; d < D; d += kTailThreads) {
      double sk = 0.0, sv = 0.0;
      for (int r = 0; r < RPS; ++r) {
        sk += redk[r][d];
        sv += redv[r][d];
      }
      kpart_out[((u * nsplit + split) * 2 + 0) * D + d] = sk;
      kpart_out[((u * nsplit + split) * 2 + 1) * D + d] = sv;
    }
  }
}

// Per unit: combine partials, form the slot, append it to the packed cache.
template <int D, typename T, bool DO_TAIL, bool DO_COMPACT>
__global__ __launch_bounds__(kTailThreads) void tail_finalize_kernel(
    Geo g, SeqTab st, int32_t nsplit, int32_t nslice, const int64_t* __restrict__ kept_offsets,
    const double* __restrict__ kpart, const double* __restrict__ mpart,
    const double* __restrict__ evicted_sum, const double* __restrict__ total_sum,
    const double* __restrict__ ksum, const double* __restrict__ vsum, float* __restrict__ k_star,
    float* __restrict__ v_star, double* __restrict__ tail_mass, T* __restrict__ k_packed,
    T* __restrict__ v_packed, int32_t* __restrict__ pos_packed) {
  __shared__ float slot_k[D], slot_v[D];

  const int h = blockIdx.x % g.H;
  const int bl = blockIdx.x / g.H;
  const int l = blockIdx.y;
  if (bl >= st.count) return;
  const int b = st.first + bl;
  const int n = st.len[bl];
  const int64_t u = unit_index(g, l, b, h);
  const int tid = threadIdx.x;
  const int64_t off = kept_offsets[u];
  const int nk = (int)(kept_offsets[u + 1] - off);

  if (DO_TAIL) {
    const TailMass tm = tail_masses(u, n, nk, nslice, ksum && vsum, evicted_sum, total_sum, mpart);
    const int per = GatherStep<D, T>::rows(nk, nsplit);
    const int used = tm.direct ? nsplit : (nk + per - 1) / per;  // the partials that were written
    for (int x = tid; x < 2 * D; x += kTailThreads) {
      // x: a key dimension, or D + a value dimension
      double sum = 0.0;
      // partials added in split order, the loads of 32 splits in flight together
      // (those past the last read it again and are not added)
      for (int s0 = 0; s0 < used; s0 += 32) {
        double y[32];
#pragma unroll
        for (int i = 0; i < 32; ++i)
          y[i] = kpart[(u * nsplit + min(s0 + i, used - 1)) * 2 * D + x];
#pragma unroll
        for (int i = 0; i < 32; ++i) sum += s0 + i < used ? y[i] : 0.0;
      }
      const int d = x < D ? x : x - D;
      if (!tm.direct) sum = (x < D ? ksum : vsum)[u * D + d] - sum;
      (x < D ? slot_k : slot_v)[d] = tm.ev > 0.0 ? (float)(sum / tm.ev) : 0.f;
    }
    __syncthreads();
    for (int d = tid; d < D; d += kTailThreads) {
      k_star[u * D + d] = slot_k[d];
      v_star[u * D + d] = slot_v[d];
    }
    if (tid == 0) tail_mass[u] = tm.ev / tm.all;
  } else {
    for (int d = tid; d < D; d += kTailThreads) {
      slot_k[d] = k_star[u * D + d];
      slot_v[d] = v_star[u * D + d];
    }
    __syncthreads();
  }
  if (DO_COMPACT && g.slot) {
    const int64_t prow = off + u + nk;
    for (int d = tid; d < D; d += kTailThreads) {
      k_packed[prow * D + d] = from_f32<T>(slot_k[d]);
      v_packed[prow * D + d] = from_f32<T>(slot_v[d]);
    }
    if (tid == 0) pos_packed[prow] = -1;
  }
}

template <int D, typename T, bool DT, bool DC>
static certkv_status launch_tail(const TailArgs& a, const SeqTab& st, hipStream_t s) {
  const Geo& g = a.g;
  const dim3 grid_split(g.H * st.count * a.nsplit, g.L);
  const dim3 grid_slice(g.H * st.count * a.nslice, g.L);
  const dim3 grid_unit(g.H * st.count, g.L);
  const char* gname = DT ? (DC ? "tail_compact_gather" : "tail_gather") : "compact_gather";
  const char* fname = DT ? (DC ? "tail_compact_finalize" : "tail_finalize") : "compact_slot";
  if (DT && !(a.evicted_sum && a.total_sum))
    CERTKV_LAUNCH("tail_mass", mass_kernel, grid_slice, dim3(kTailThreads), 0, s, g, st, a.nslice,
                  a.scores, (const uint64_t*)a.bitmap, a.bm_stride, a.mpart);
  CERTKV_LAUNCH(gname, (tail_gather_kernel<D, T, DT, DC>), grid_split, dim3(kTailThreads), 0, s, g,
                st, a.nsplit, a.nslice, a.ksum && a.vsum, (const uint64_t*)a.bitmap, a.bm_stride,
                (const double*)a.mpart, a.evicted_sum, a.total_sum, a.scores,
                static_cast<const T*>(a.k.ptr), a.k.s_layer, a.k.s_token, a.k.s_head,
                static_cast<const T*>(a.v.ptr), a.v.s_layer, a.v.s_token, a.v.s_head,
                a.kept_offsets, a.kept_idx, a.kpart, static_cast<T*>(a.k_packed),
                static_cast<T*>(a.v_packed), a.pos_packed);
  CERTKV_LAUNCH(fname, (tail_finalize_kernel<D, T, DT, DC>), grid_unit, dim3(kTailThreads), 0, s, g,
                st, a.nsplit, a.nslice, a.kept_offsets, (const double*)a.kpart, (const double*)a.mpart,
                a.evicted_sum, a.total_sum, a.ksum, a.vsum, a.k_star, a.v_star, a.tail_mass,
                static_cast<T*>(a.k_packed), static_cast<T*>(a.v_packed), a.pos_packed);
  return CERTKV_OK;
}

template <int D, typename T>
static certkv_status dispatch_tail(const TailArgs& a, const SeqTab& st, hipStream_t s) {
  if (a.do_tail && a.do_compact) return launch_tail<D, T, true, true>(a, st, s);
  if (a.do_tail) return launch_tail<D, T, true, false>(a, st, s);
  return launch_tail<D, T, false, true>(a, st, s);
}

certkv_status run_bitmap(const TailArgs& a, const SeqTab& st, int64_t words_total, bool clear,
                         hipStream_t s) {
  if (clear)
    CERTKV_LAUNCH("kept_bitmap_clear", bitmap_clear_kernel, dim3((unsigned)((words_total + 255) / 256)),
                  dim3(256), 0, s, a.bitmap, words_total);
  CERTKV_LAUNCH("kept_bitmap_set", bitmap_set_kernel,
                dim3(a.g.H * st.count * a.nsplit, a.g.L), dim3(256), 0, s, a.g, st, a.nsplit, a.kept_offsets, a.kept_idx, a.bitmap, a.bm_stride);
  return CERTKV_OK;
}

certkv_status run_tail(const TailArgs& a, const SeqTab& st, hipStream_t s) {
  if (a.dtype == CERTKV_BF16)
    return a.g.D == 128 ? dispatch_tail<128, uint16_t>(a, st, s) : dispatch_tail<64, uint16_t>(a, st, s);
  return a.g.D == 128 ? dispatch_tail<128, float>(a, st, s) : dispatch_tail<64, float>(a, st, s);
}

}  // namespace certkv
