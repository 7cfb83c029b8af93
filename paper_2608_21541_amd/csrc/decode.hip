// Decode over the packed cache on gfx950.
//
// After the pass each head keeps its b_h real rows and one charged slot row
// (k*, v*) (Section 4.1); a later query attends over these rows as ordinary
// keys, the plain slot carrying no logit bias.  For the tq new queries of a
// sequence and KV head h, the M = tq * G query rows (row = t * G + g) attend
// over the unit's packed segment:
//   z_i = scale <q, k_i>,  out = sum_i softmax(z)_i v_i,  lse = log sum e^z.
//
// Split over keys: the packed rows are cut into chunks of the same length
// (dec_cut), one or so for each of the workgroups that stay resident; a
// workgroup finds the units of its chunk in the packed offsets.  A workgroup holds the unit's query tiles of
// 32 rows, one wave each; with fewer than four tiles, two or four waves share
// a tile and split its output dims.  Key and value tiles of 32 rows go from
// memory straight into LDS (wave-wide 16-byte LDS-DMA loads into a ring of
// five tile buffers, XOR-swizzled chunks, rows in natural order).  Per tile
// and wave:
//   S^T = K Q^T on v_mfma_f32_32x32x16_bf16 with the key tile as the A
//     operand, so lane (hh, c) holds query row c and 16 of the tile's keys;
//   online softmax in log2 units, the row maximum shared by the two lanes of
//     a row, the accumulators rescaled only when a row maximum grows by more
//     than 2^8 (weights stay below 2^8, the partial is unchanged);
//   O^T += V^T P^T on the same MFMA: P^T (B operand) comes straight from the
//     lane's registers, split into a bf16 high part and the bf16 of the
//     remainder (two MFMAs, about 16 bits of the fp32 weight), and V^T (A
//     operand) comes from transposing LDS reads of the key-major value tile
//     along the same key order.
// The partials (reference max, sum, unnormalized output) are combined in row
// order by a second kernel (deterministic).
#include "stages.h"

namespace certkv {

constexpr int kDecTileShift = 5;
constexpr int kDecTile = 1 << kDecTileShift;  // keys per tile
constexpr int kDecSumShift = 12;  // 4096 keys per fp32 accumulator

typedef __bf16 dec_bf16x8 __attribute__((__vector_size__(8 * sizeof(__bf16))));
typedef float dec_f32x16 __attribute__((__vector_size__(16 * sizeof(float))));

union DecFrag {
  uint4 u;
  uint16_t h[8];
  dec_bf16x8 v;
};

constexpr float kDecLog2e = 1.4426950408889634f;
constexpr float kDecLn2 = 0.6931471805599453f;
constexpr float kDecSlack = 8.f;  // log2 growth of the row maximum absorbed without rescaling

typedef __bf16 dec_bf16x2 __attribute__((ext_vector_type(2)));
typedef float dec_f32x2 __attribute__((ext_vector_type(2)));

// Two floats to bf16 (round to nearest even), a in the low half.
__device__ __forceinline__ uint32_t dec_pack_bf16(float a, float b) {
  const dec_bf16x2 h = __builtin_convertvector((dec_f32x2){a, b}, dec_bf16x2);
  return __builtin_bit_cast(uint32_t, h);
}


// 16 bytes at addresses aligned to an element only: the caller's cluster summaries
// and outputs (a row count or an offset of its own may come before them).
typedef uint32_t dec_u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
typedef float dec_f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ uint4 dec_load_any(const uint16_t* p) {
  const dec_u32x4_any x = *reinterpret_cast<const dec_u32x4_any*>(p);
  return make_uint4(x[0], x[1], x[2], x[3]);
}

// Workgroup shape: every wave takes one 32-row query tile and all keys; with
// fewer than four query tiles, DS waves share a query tile and split the
// output dims (each computes the tile's scores and softmax, and P V for its
// D / DS dims), down to 32 dims per wave.
template <int D, int NQT>
struct DecShape {
  static constexpr int DS0 = NQT >= 4 ? 1 : 4 / NQT;
  static constexpr int DS = DS0 < D / 32 ? DS0 : D / 32;  // dim splits per query tile
  static constexpr int NW = NQT * DS;                      // waves per workgroup
  static constexpr int NDBW = D / 32 / DS;                 // 32-dim blocks per wave
};

// LDS pipeline: a stage is one key tile (K and V); NBUF stage buffers, up to
// kDecLdsBytes and at most five (two workgroups per compute unit).
constexpr int kDecLdsBytes = 80 * 1024;
template <int D>
struct DecPipe {
  static constexpr int STAGE_BYTES = 2 * kDecTile * D * 2;
  static constexpr int NB0 = kDecLdsBytes / STAGE_BYTES;
  static constexpr int NBUF = NB0 > 5 ? 5 : NB0;
  static_assert(NBUF >= 3, "three stage buffers at least");
};

// LDS layout of a stage: [tile][K, V][32 rows][D/8 chunks of 16 bytes], rows
// in natural (key-major) order.  Chunks are XOR-swizzled within a row so that
// both fragment reads are free of bank conflicts: the key-tile read (one
// 16-byte chunk per lane, 16 consecutive rows per pass) and the transposing
// value-tile read (8 bytes per lane, four consecutive rows and eight
// consecutive 32-byte segments per half-wave).  The map is an involution:
// the slot of chunk c is c ^ f(r) and the chunk in slot s is s ^ f(r).
template <int D>
__device__ __forceinline__ int dec_swz_k(int r, int c) {
  return c ^ ((D == 128 ? r : (r >> 1)) & (D / 8 - 1));
}
template <int D>
__device__ __forceinline__ int dec_swz_v(int r, int c) {
  return c ^ (D == 128 ? 4 * (r & 3) : 4 * ((r >> 1) & 1));
}

// One wave-wide 16-byte load straight into LDS: lane L's 16 bytes from src
// land at LDS byte address lds + 16 L (lds wave-uniform, through M0).  Issued
// as inline assembly so that the compiler does not treat the load as a
// pending LDS write (which would make it wait for every load in flight at
// each barrier); the caller waits for it with dec_wait_vm0 before the
// barrier that publishes the stage.  Non-temporal: a row is read once per call
// (32 layers, 3.36M rows, one query: 338 us without, 5.1 TB/s; 287 with).
__device__ __forceinline__ void dec_dma16(const void* src, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt"
               :
               : "v"(src), "s"(__builtin_amdgcn_readfirstlane(lds))
               : "memory", "m0");
}

// Wait until at most N vector-memory accesses of this wave are in flight
// (the other counters at their maximum; a builtin, so the compiler's own
// bookkeeping of outstanding loads sees it).
template <int N>
__device__ __forceinline__ void dec_wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
__device__ __forceinline__ void dec_wait_vm0() { dec_wait_vm<0>(); }

// dec_wait_vm<PER * n> for a wave-uniform n in [0, NMAX].
template <int PER, int NMAX>
__device__ __forceinline__ void dec_wait_stages(int n) {
  if constexpr (NMAX == 0) {
    dec_wait_vm<0>();
  } else {
    if (n >= NMAX)
      dec_wait_vm<PER * NMAX>();
    else
      dec_wait_stages<PER, NMAX - 1>(n);
  }
}

__device__ __forceinline__ uint32_t dec_lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

typedef short dec_s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) dec_s16x4 dec_lds_s16x4;

// The packed rows of all units, one after another, are cut into as many chunks
// of the same length as workgroups are resident at once, so that every one gets the
// same share however the rows are spread over the units: a chunk that crosses from
// one unit to the next is two pieces.  Microseconds with chunks of 4096 keys cut
// per unit, and so: 32 layers of 8 heads, 3.36M rows, one query 363 and 278; 12
// layers of three sequences, 144 units, 618k rows 109 and 70; 7 layers of eight,
// 896 units of 64 dims, 722k rows, 32 query rows 151 and 81; one layer of 26216 rows, in
// 128-key chunks, the shortest, 105 and 15.
// Chunks depend on the rows of the whole call, so a row's sums are grouped, and
// rounded, differently beside other units.
// A piece longer than 4096 rows writes a partial for every 4096 of them, the
// bound on how long an fp32 sum gets (3.36M rows, sums of up to 6592: errors against
// 64 bits 0.2 to 0.4 % larger), while its loads run on: in two chunks one after the
// other, with the loads drained between them, the same rows take 5 % longer.
// (Rows are counted in 32 bits, which divide in a few instructions: 2^31 rows of 64
// dims are 512 GB.)
struct DecCut {
  uint32_t keys;  // rows per chunk
  int sum_shift;  // log2 of the rows per partial
  // partials of that many rows of one piece
  __device__ __forceinline__ uint32_t partials(uint32_t rows) const {
    return (rows + (1u << sum_shift) - 1u) >> sum_shift;
  }
};
__device__ __forceinline__ DecCut dec_cut(const DecodeChunks& c, uint32_t rows, int64_t U) {
  // With few rows the fixed cost of a piece (its queries, first tile and partials)
  // outweighs them.  Then the chunks are fewer by the units' starts, so that every
  // piece is a workgroup's only one: two of them per compute unit up to 1024 keys
  // each, one up to 512 where the units are few (128 units of 64 dims, 131k rows, 64
  // query rows: chunks of 128, 160, 352 keys 40, 41, 33 us; 32 units of 128 dims,
  // 105k rows 41 us in chunks of 224, 34 of 480; of 1676 keys, 144 units: 70 us in
  // 512 chunks, 76 in 369).
  // (From the rows and not from the caller's bound on them: the chunks, and so the
  // bits, are the same under any bound.)
  constexpr uint32_t kOne = 256, kTwo = 512;
  const uint32_t two = min((uint32_t)c.parts, kTwo);
  uint32_t n = (uint32_t)c.parts;
  if (n > kOne && 4 * U <= kOne && rows <= (kOne - (uint32_t)U + 1u) * 512u)
    n = kOne - (uint32_t)U + 1u;
  else if (2 * U <= two && rows <= (two - (uint32_t)U + 1u) * 1024u)
    n = two - (uint32_t)U + 1u;
  uint32_t k = rows <= n * (uint32_t)c.keys_min ? (uint32_t)c.keys_min : (rows + n - 1u) / n;
  // (more rows than the bound allows for: longer chunks and sums, so that the
  // partials stay within the workspace)
  if (rows > (uint64_t)c.most * k) k = (rows + (uint32_t)c.most - 1u) / (uint32_t)c.most;
  DecCut cut{(k + kDecTile - 1u) & ~(uint32_t)(kDecTile - 1), kDecSumShift};
  while ((rows >> cut.sum_shift) > (uint32_t)c.sums) ++cut.sum_shift;
  return cut;
}

// Partials: those of a unit lie one after the other, its first at this place,
// where s0 is the chunk of its first row, `at` rows after the first unit's.  A unit
// of len rows has a piece for each of its chunks and at most len >> sum_shift
// partials beyond one for each, so that it ends before the next one's place.
__device__ __forceinline__ uint32_t dec_place(const DecCut& cut, uint32_t at, uint32_t s0,
                                              uint32_t u) {
  return (at >> cut.sum_shift) + s0 + u;
}
// Rows of the first piece of a unit of len rows.
__device__ __forceinline__ uint32_t dec_first(const DecCut& cut, uint32_t at, uint32_t s0,
                                              uint32_t len) {
  return min(len, (s0 + 1u) * cut.keys - at);
}
// Partials of a unit whose first len rows are attended.
__device__ __forceinline__ uint32_t dec_partials(const DecCut& cut, uint32_t at, uint32_t s0,
                                                 uint32_t len) {
  const uint32_t first = dec_first(cut, at, s0, len), rest = len - first;
  if (rest == 0) return cut.partials(first);
  const uint32_t whole = rest / cut.keys;
  return cut.partials(first) + whole * cut.partials(cut.keys) +
         cut.partials(rest - whole * cut.keys);
}

// x of lane i (wave-uniform).
__device__ __forceinline__ int64_t dec_readlane(int64_t x, int i) {
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)x, i);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)((uint64_t)x >> 32), i);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The unit that holds packed row r (counted from the first unit's), by a wave:
// 64 units' ends per step.  U past the last row.
__device__ __forceinline__ int dec_find_unit(const int64_t* __restrict__ poff, int U, int64_t r,
                                             int lane) {
  int lo = 0, n = U;  // the answer is one of [lo, lo + n]
  while (true) {
    const int step = (n + 63) / 64;
    const int i = lo + lane * step + step - 1;
    const bool past = i >= U || poff[i + 1] - poff[0] > r;  // unit i ends past r
    lo += (int)__popcll(__ballot(!past)) * step;
    if (step == 1) return min(lo, U);
    n = step;
  }
}

template <int D, int NQT>
__device__ __forceinline__ void decode_body(
    const Geo& g, int64_t U, const DecodeChunks& ck, int32_t tq, int32_t mp,
    const uint16_t* __restrict__ qn, int64_t q_sl, int64_t q_st, int64_t q_sh,
    const uint16_t* __restrict__ kp, const uint16_t* __restrict__ vp,
    const int64_t* __restrict__ poff, float* __restrict__ part_o, float2* __restrict__ part_ml) {
  constexpr int NW = DecShape<D, NQT>::NW;
  constexpr int NDBW = DecShape<D, NQT>::NDBW;
  constexpr int NBUF = DecPipe<D>::NBUF;
  constexpr int KS = D / 16;       // MFMA k-steps of S^T
  constexpr int HD = D / 2;        // dims per lane half in S^T
  constexpr int CH = D / 8;        // 16-byte chunks per row
  constexpr int TILE = kDecTile * D;          // bf16 elements of one K (or V) tile
  constexpr int TILE_CH = kDecTile * CH;      // its 16-byte chunks
  constexpr int NINS = 2 * TILE_CH / 64;      // wave-wide 16-byte loads per stage
  constexpr int PERW = NINS >= NW ? NINS / NW : 1;  // of them per wave (or none)
  static_assert((NINS % NW == 0 || NINS < NW) && TILE_CH % 64 == 0, "stage split");
  __shared__ __align__(16) uint16_t lds[NBUF][2][TILE];

  // A persistent grid over the chunks, and in each over the units it meets.
  // Up to 64 units: their segments in the lanes of every wave, so that a piece
  // waits for one load before its queries and tiles, not for three in turn.
  // (Not with eight query tiles and more, whose registers are all taken.)
  const bool few = NQT < 8 && U <= 64;
  const int lane = threadIdx.x & 63;
  int64_t ps = 0, pe = 0;
  if (few) {
    ps = poff[min(lane, (int)U)];
    pe = poff[min(lane + 1, (int)U)];
  }
  auto seg_start = [&](int64_t u) { return few ? dec_readlane(ps, (int)u) : poff[u]; };
  auto seg_end = [&](int64_t u) { return few ? dec_readlane(pe, (int)u) : poff[u + 1]; };
  const int64_t base = seg_start(0), rows = seg_end(U - 1) - base;
  const DecCut cut = dec_cut(ck, (uint32_t)rows, U);
  const int keys = (int)cut.keys;
  // Where the grid has workgroups left for the units' first pieces, those that
  // start inside a chunk are theirs, and no workgroup takes two pieces in turn.
  const int64_t nch = ((uint32_t)rows + cut.keys - 1u) / cut.keys;
  const bool heads = nch + U - 1 <= gridDim.x;
  for (int64_t x = blockIdx.x; x < (heads ? nch + U - 1 : nch); x += gridDim.x) {
  const int64_t head = x - nch + 1;  // from 1: the unit whose first piece is taken
  const int64_t r0 = x < nch ? x * keys : seg_start(head) - base;
  const int64_t s = x < nch ? x : (uint32_t)r0 / cut.keys, r1 = min(rows, (s + 1) * keys);
  if (x >= nch && r0 == s * keys) continue;  // a chunk's first piece
  const uint64_t past = __ballot(pe - base > r0);
  const int64_t u0 = x >= nch ? head
                     : few    ? (past ? (int64_t)__builtin_ctzll(past) : U)
                              : dec_find_unit(poff, (int)U, r0, lane);
  for (int64_t u = u0; u < U; u = heads ? U : u + 1) {
  const int64_t p0 = seg_start(u), at = p0 - base;  // the unit's first row, and from the first unit's
  if (at >= r1) break;
  const int len = (int)(seg_end(u) - p0);
  const int c0 = (int)max(r0 - at, (int64_t)0);
  const int c1 = (int)min(min(ck.cover, (int64_t)len), r1 - at);
  if (c0 >= c1) continue;  // whole workgroup: an empty unit, or rows past the caller's bound
  const int h = (int)(u % g.H);
  const int64_t lb = u / g.H;
  const int b = (int)(lb % g.B);
  const int l = (int)(lb / g.B);
  const int ntiles = (c1 - c0 + kDecTile - 1) / kDecTile;
  const int M = tq * g.G;
  const int wave = threadIdx.x >> 6;
  const int qt = wave % NQT;        // query tile of this wave
  const int dsi = wave / NQT;       // its share of the output dims
  const int db0 = dsi * NDBW;       // first 32-dim block of that share
  const int hh = lane >> 5;
  const int c32 = lane & 31;
  const int row = qt * 32 + c32;    // this lane's query row
  const float c2 = g.scale * kDecLog2e;

  // A stage goes from memory straight into LDS: wave-wide 16-byte loads, lane
  // L of load n filling chunk slot 64 n + L of the stage.  The chunk a slot
  // holds is chosen by the swizzle; rows past the segment are clamped to its
  // last row (their keys are masked, so they only ever meet zero weights).
  const uint16_t* kseg = kp + p0 * D;
  const uint16_t* vseg = vp + p0 * D;
  auto issue_stage = [&](int st) {
#pragma unroll
    for (int i = 0; i < PERW; ++i) {
      const int n = wave * PERW + i;
      const int kv = n / (TILE_CH / 64);                    // uniform over the wave
      if (n < NINS) {
        const int pos = (n % (TILE_CH / 64)) * 64 + lane;   // slot within the tile
        const int r = pos / CH;
        const int chunk = kv ? dec_swz_v<D>(r, pos % CH) : dec_swz_k<D>(r, pos % CH);
        const int key = min(c0 + st * kDecTile + r, len - 1);
        const uint16_t* src = (kv ? vseg : kseg) + (int64_t)key * D + chunk * 8;
        dec_dma16(src, dec_lds_addr(&lds[st % NBUF][kv][(n % (TILE_CH / 64)) * 512]));
      }
    }
  };

  DecFrag qf[KS];
  float m_run, l_run;
  dec_f32x16 O[NDBW];  // O^T of the wave's 32-dim blocks db0 ..

  // S^T = K Q^T of the key tile in stage buffer sb: lane (hh, c32) holds
  // query row c32 and keys 8*(v/4) + 4*hh + v%4 of the tile.
  auto score_tile = [&](int sb) {
    const uint16_t* kt = lds[sb][0];
    dec_f32x16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      DecFrag kf;
      kf.u = *reinterpret_cast<const uint4*>(kt + c32 * D +
                                             dec_swz_k<D>(c32, hh * (CH / 2) + ks) * 8);
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf.v, qf[ks].v, s, 0, 0, 0);
    }
    return s;
  };

  // Softmax and O^T += V^T P^T of the tile (first key t0) whose scores are s.
  auto finish_tile = [&](int sb, int t0, dec_f32x16 s) {
    const uint16_t* vt = lds[sb][1];
    // Online softmax of the row in log2 units (z = c2 * s, c2 > 0, so the
    // maximum is taken on the raw products).  Keys past the chunk occur only
    // in its last tile.
    if (t0 + kDecTile > c1) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int key = t0 + 8 * (v >> 2) + 4 * hh + (v & 3);
        s[v] = key < c1 ? s[v] : -INFINITY;
      }
    }
    float mt = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mt = fmaxf(mt, s[v]);
    {
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mt), __float_as_uint(mt),
                                                       false, false);
      mt = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * c2;
    }
    // Lazy rescaling: the reference maximum m_run moves only when some row of
    // the wave would otherwise see a weight above 2^kDecSlack; the weights
    // exp2(z - m_run) then stay below 2^kDecSlack and the partial (m_run,
    // l_run, O) is the same quantity for any reference.
    if (__builtin_amdgcn_ballot_w64(mt > m_run + kDecSlack) != 0) {
      const float mnew = fmaxf(m_run, mt);
      const float alpha = __builtin_amdgcn_exp2f(m_run - mnew);
      m_run = mnew;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < NDBW; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) O[db][v] *= alpha;
    }
    // P^T fragments: k-step kk takes the lane's values v = 8 kk .. 8 kk + 7,
    // i.e. keys 16 kk + 8 (i/4) + 4 hh + i%4 for k-slot 8 hh + i; each weight
    // is the bf16 (round to nearest even) of p plus the bf16 of p - hi.
    DecFrag ph[2], pl[2];
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      const float p0 = __builtin_amdgcn_exp2f(fmaf(s[v], c2, -m_run));
      const float p1 = __builtin_amdgcn_exp2f(fmaf(s[v + 1], c2, -m_run));
      l_run += p0 + p1;
      const uint32_t hi = dec_pack_bf16(p0, p1);
      const float r0 = p0 - __uint_as_float(hi << 16);
      const float r1 = p1 - __uint_as_float(hi & 0xffff0000u);
      reinterpret_cast<uint32_t*>(&ph[v >> 3].u)[(v & 7) >> 1] = hi;
      reinterpret_cast<uint32_t*>(&pl[v >> 3].u)[(v & 7) >> 1] = dec_pack_bf16(r0, r1);
    }
    // O^T += V^T P^T per 32-dim block.  V^T (A operand): lane (hh, c32) needs
    // dim 32 db + c32 at the keys of its k-slots.  A transposing read serves
    // them from the key-major tile: in each group of 16 lanes, lane a
    // addresses key 16 kk + 8 rd + 4 hh + a/4 at dims 4 (a%4) .. 4 (a%4) + 3
    // of its group's 16 dims, and lane i receives dim i of keys
    // 16 kk + 8 rd + 4 hh + 0..3, which are its k-slots 4 rd .. 4 rd + 3.
    const int a = c32 & 15;
    const int vdim = 16 * (c32 >> 4) + 4 * (a & 3);  // + 32 db
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int db = 0; db < NDBW; ++db) {
        DecFrag vf;
#pragma unroll
        for (int rd = 0; rd < 2; ++rd) {
          const int r = 16 * kk + 8 * rd + 4 * hh + (a >> 2);
          const int dim = 32 * (db0 + db) + vdim;
          const uint16_t* src = vt + r * D + dec_swz_v<D>(r, dim >> 3) * 8 + (dim & 7);
          const dec_s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (dec_lds_s16x4*)(__attribute__((address_space(3))) uint16_t*)src);
          reinterpret_cast<uint2*>(&vf.u)[rd] = __builtin_bit_cast(uint2, x);
        }
        O[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf.v, ph[kk].v, O[db], 0, 0, 0);
        O[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf.v, pl[kk].v, O[db], 0, 0, 0);
      }
    }
  };

  // Stage 0 and the query fragments are awaited together; then stages up to
  // NBUF - 2 ahead of the one consumed are in flight.  Before stage st each
  // wave waits until its own loads of st have landed (loads complete in
  // order, so those of the later stages already issued may stay in flight);
  // the barrier then publishes stage st and certifies that every wave is done
  // with stage st - 1, whose buffer the loads of stage st + NBUF - 1
  // overwrite.
  issue_stage(0);
  // The query row as B fragments of S^T (zero for padding rows); lane half hh
  // owns the dims hh*HD .. hh*HD + HD - 1 (the contraction order is free).
  if (row < M) {
    const int t = row / g.G, gq = row % g.G;
    const uint4* src = reinterpret_cast<const uint4*>(
        qn + (int64_t)l * q_sl + (int64_t)(b * tq + t) * q_st + (int64_t)(h * g.G + gq) * q_sh +
        hh * HD);
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[s].u = src[s];
  } else {
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[s].u = make_uint4(0u, 0u, 0u, 0u);
  }

  // the place of the piece's first partial
  const uint32_t s0 = (uint32_t)at / cut.keys;
  uint32_t place = dec_place(cut, (uint32_t)at, s0, (uint32_t)u);
  if (s > s0)
    place += cut.partials(dec_first(cut, (uint32_t)at, s0, (uint32_t)len)) +
             ((uint32_t)s - s0 - 1u) * cut.partials(cut.keys);

  dec_wait_vm0();
  for (int st = 1; st < NBUF - 1 && st < ntiles; ++st) issue_stage(st);
  for (int st = 0; st < ntiles;) {
    // the rows of one partial
    const int st0 = st, st_end = min(ntiles, st + (1 << (cut.sum_shift - kDecTileShift)));
    m_run = -INFINITY;
    l_run = 0.f;
#pragma unroll
    for (int db = 0; db < NDBW; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) O[db][v] = 0.f;
    for (; st < st_end; ++st) {
      dec_wait_stages<PERW, NBUF - 2>(min(NBUF - 2, ntiles - 1 - st));
      __syncthreads();
      if (st + NBUF - 1 < ntiles) issue_stage(st + NBUF - 1);
      finish_tile(st % NBUF, c0 + st * kDecTile, score_tile(st % NBUF));
    }
    // the row's (max, sum), from the first wave of the query tile (every wave of
    // it holds the same), and the unnormalized output of each wave's dims
    const float l_row = l_run + __shfl_xor(l_run, 32, 64);
    const int64_t pr =
        (int64_t)(place + ((uint32_t)st0 >> (cut.sum_shift - kDecTileShift))) * mp + row;
    if (row < M) {  // (the tile's padding rows are not written)
      if (dsi == 0 && hh == 0) part_ml[pr] = make_float2(m_run, l_row);
      float* po = part_o + pr * D;
#pragma unroll
      for (int db = 0; db < NDBW; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          po[32 * (db0 + db) + 8 * (v >> 2) + 4 * hh + (v & 3)] = O[db][v];
    }
  }
  __syncthreads();  // every wave is done with the stage buffers of this piece
  }
  }
}

// Two waves per SIMD at least: the register cap keeps the accumulators out of
// AGPRs; three where three workgroups fit a compute unit (decode_parts).
template <int D, int NQT>
__global__ __launch_bounds__((64 * DecShape<D, NQT>::NW))
__attribute__((amdgpu_waves_per_eu(D == 64 && NQT == 4 ? 3 : 2))) void decode_kernel(
    Geo g, int64_t U, DecodeChunks ck, int32_t tq, int32_t mp, const uint16_t* __restrict__ qn, int64_t q_sl, int64_t q_st, int64_t q_sh,
    const uint16_t* __restrict__ kp, const uint16_t* __restrict__ vp,
    const int64_t* __restrict__ poff, float* __restrict__ part_o, float2* __restrict__ part_ml) {
  decode_body<D, NQT>(g, U, ck, tq, mp, qn, q_sl, q_st, q_sh, kp, vp, poff, part_o, part_ml);
}

// Combine the chunk partials of each (unit, row): one workgroup per row, the
// partial slots dealt round-robin to groups of D/4 threads (four output dims
// per thread, 16-byte loads).  Each group folds its slots in order with an
// online maximum; the groups are then merged in group order through LDS, so
// the result does not depend on timing.
constexpr int kCombThreads = 256;

// With clustered tail summaries (CL), the m cluster terms n_g e^{lbar_g}
// (lbar_g = scale <q, kbar_g>) and n_g e^{lbar_g} vbar_g join the kept rows'
// sums (the ratio estimator of the clustered-summary bound), and the row's
// runtime certificate is evaluated from the stored summaries, a cluster to a
// lane (two layers, 16 clusters, 16 rows a head: 20 us with the dot products
// and the certificate one cluster after the other, 11 us): with r_g =
// scale |q| R_g and zeta_g = n_g e^{lbar_g} / Zhat,
//   D_Z / Zhat = sum_g (e^r_g - 1) e^r_g zeta_g,
//   D_N / Zhat = sum_g e^r_g zeta_g ((e^r_g - 1) |vbar_g| + rho_g),
//   V' = max(max kept |v|, max_g |vbar_g| + rho_g),
// and |Ohat - O| <= 3 (D_N + V' D_Z) / Zhat when D_Z <= Zhat / 3 (else the
// bound is infinite).
template <int D, bool CL>
__global__ __launch_bounds__(kCombThreads) void decode_combine_kernel(
    Geo g, int64_t U, DecodeChunks ck, int32_t tq, int32_t mp, const int64_t* __restrict__ poff,
    const float* __restrict__ part_o,
    const float2* __restrict__ part_ml, float* __restrict__ out, float* __restrict__ lse,
    DecodeClusters cl, const uint16_t* __restrict__ qn, int64_t q_sl,
    int64_t q_st, int64_t q_sh) {
  constexpr int kMaxCl = 64;
  __shared__ float zc_s[CL ? kMaxCl : 1], vn_s[CL ? kMaxCl : 1], wc_s[CL ? kMaxCl : 1];
  __shared__ float qn_s;
  constexpr int C4 = D / 4;                // threads per slot row
  constexpr int S = kCombThreads / C4;     // slot groups
  __shared__ float4 acc_s[S][C4];
  __shared__ float2 ml_s[S];
  const int64_t u = blockIdx.x;
  const int row = blockIdx.y;
  const int sg = threadIdx.x / C4;
  const int c4 = threadIdx.x % C4;
  const int len = (int)(poff[u + 1] - poff[u]);
  const DecCut cut = dec_cut(ck, (uint32_t)(poff[U] - poff[0]), U);
  const uint32_t at_row = (uint32_t)(poff[u] - poff[0]), s0 = at_row / cut.keys;
  const int nv = (int)dec_partials(cut, at_row, s0, (uint32_t)min(ck.cover, (int64_t)len));
  const int64_t base = (int64_t)dec_place(cut, at_row, s0, (uint32_t)u) * mp + row;  // + slot * mp
  if (len > ck.cover && row == 0 && threadIdx.x == 0) report_range(g);
  float m = -INFINITY, L = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  auto fold = [&](float2 ml, float4 o) {
    if (ml.x == -INFINITY) return;
    if (ml.x > m) {
      const float a = __builtin_amdgcn_exp2f(m - ml.x);  // 0 while m is -inf
      L *= a;
      acc.x *= a; acc.y *= a; acc.z *= a; acc.w *= a;
      m = ml.x;
    }
    const float w = __builtin_amdgcn_exp2f(ml.x - m);
    L += ml.y * w;
    acc.x += o.x * w; acc.y += o.y * w; acc.z += o.z * w; acc.w += o.w * w;
  };
  int sp = sg;
  for (; sp + 3 * S < nv; sp += 4 * S) {  // four slots in flight
    float2 ml[4];
    float4 o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t pr = base + (int64_t)(sp + i * S) * mp;
      ml[i] = part_ml[pr];
      o[i] = reinterpret_cast<const float4*>(part_o + pr * D)[c4];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) fold(ml[i], o[i]);
  }
  for (; sp < nv; sp += S) {
    const int64_t pr = base + (int64_t)sp * mp;
    fold(part_ml[pr], reinterpret_cast<const float4*>(part_o + pr * D)[c4]);
  }
  acc_s[sg][c4] = acc;
  if (c4 == 0) ml_s[sg] = make_float2(m, L);
  const int Hq = g.H * g.G;
  const int h = (int)(u % g.H);
  const int64_t lb = u / g.H;
  const int b = (int)(lb % g.B);
  const int l = (int)(lb / g.B);
  const int t = row / g.G, gq = row % g.G;
  const int64_t orow = ((int64_t)l * g.B * tq + (int64_t)b * tq + t) * Hq + h * g.G + gq;
  const float c2 = g.scale * kDecLog2e;
  if (CL) {
    // cluster logits in log2 units (with log2 n_g) and value norms: D / 8 lanes
    // per cluster, 8 dims each
    constexpr int LC = D / 8;
    const uint4 qv = reinterpret_cast<const uint4*>(
        qn + (int64_t)l * q_sl + (int64_t)(b * tq + t) * q_st +
        (int64_t)(h * g.G + gq) * q_sh)[threadIdx.x % LC];
    auto at8 = [](const uint4& x, int e) {
      const uint32_t w = (&x.x)[e >> 1];
      return e & 1 ? bf16_hi(w) : bf16_lo(w);
    };
    for (int g0 = 0; g0 < cl.m; g0 += kCombThreads / LC) {
      const int gi = min(g0 + (int)threadIdx.x / LC, cl.m - 1);
      const int64_t at = (u * cl.m + gi) * D + 8 * (threadIdx.x % LC);
      const uint4 kv = dec_load_any(cl.kbar + at), vv = dec_load_any(cl.vbar + at);
      float dot = 0.f, nv2 = 0.f, nq2 = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float qe = at8(qv, e), ve = at8(vv, e);
        dot = fmaf(qe, at8(kv, e), dot);
        nv2 = fmaf(ve, ve, nv2);
        nq2 = fmaf(qe, qe, nq2);
      }
#pragma unroll
      for (int o = LC / 2; o > 0; o >>= 1) {
        dot += __shfl_xor(dot, o, 64);
        nv2 += __shfl_xor(nv2, o, 64);
        nq2 += __shfl_xor(nq2, o, 64);
      }
      if (threadIdx.x % LC == 0 && g0 + (int)threadIdx.x / LC < cl.m) {
        const int cnt = cl.count[u * cl.m + gi];
        zc_s[gi] = cnt > 0 ? dot * c2 + __builtin_amdgcn_logf((float)cnt) : -INFINITY;
        vn_s[gi] = sqrtf(nv2);
        if (gi == 0) qn_s = sqrtf(nq2);
      }
    }
  }
  __syncthreads();
  const int dd = threadIdx.x;
  float mx = -INFINITY;
#pragma unroll
  for (int k = 0; k < S; ++k) mx = fmaxf(mx, ml_s[k].x);
  float Lt = 0.f, at = 0.f;
#pragma unroll
  for (int k = 0; k < S; ++k) {
    const float2 mk = ml_s[k];
    if (mk.x == -INFINITY) continue;
    const float w = __builtin_amdgcn_exp2f(mk.x - mx);
    Lt += mk.y * w;
    if (dd < D) at += reinterpret_cast<const float*>(&acc_s[k][0])[dd] * w;
  }
  if (CL) {
    float mc = mx;
    for (int gi = 0; gi < cl.m; ++gi) mc = fmaxf(mc, zc_s[gi]);
    const float a = mx == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mx - mc);
    Lt *= a;  // the kept rows' share, relative to 2^mc
    at *= a;
    mx = mc;
    if (dd < cl.m) wc_s[dd] = __builtin_amdgcn_exp2f(zc_s[dd] - mc);  // 0 for an empty cluster
    __syncthreads();
    for (int gi = 0; gi < cl.m; ++gi) Lt += wc_s[gi];
    if (dd < D) {
#pragma unroll 8
      for (int gi = 0; gi < cl.m; ++gi)
        at = fmaf(wc_s[gi], wc_s[gi] > 0.f ? bf16_to_f32(cl.vbar[(u * cl.m + gi) * D + dd]) : 0.f,
                    at);
    }
    if (dd < 64 && cl.bound) {
      // the certificate: a cluster per lane of the first wave
      const bool on = dd < cl.m && zc_s[dd < cl.m ? dd : 0] != -INFINITY;
      double dz = 0.0, dn = 0.0, vmax = (double)cl.vmax_kept[u];
      if (on) {
        const double rq = (double)g.scale * (double)qn_s;
        const double vn = (double)vn_s[dd], rv = (double)cl.rv[u * cl.m + dd];
        const double zeta = exp2((double)zc_s[dd] - (double)mc) / (double)Lt;
        const double er = exp(rq * (double)cl.rk[u * cl.m + dd]);
        dz = (er - 1.0) * er * zeta;
        dn = er * zeta * ((er - 1.0) * vn + rv);
        vmax = fmax(vmax, vn + rv);
      }
      dz = wave_sum(dz);
      dn = wave_sum(dn);
      vmax = wave_max(vmax);
      if (dd == 0) cl.bound[orow] = dz <= 1.0 / 3.0 ? (float)(3.0 * (dn + vmax * dz)) : INFINITY;
    }
  }
  if (dd >= D) return;
  const float o = at / Lt;
  if (!isfinite(o)) report_nonfinite(g);
  out[orow * D + dd] = o;
  if (lse && dd == 0) lse[orow] = (mx + __builtin_amdgcn_logf(Lt)) * kDecLn2;
}

// The combine for many rows: D / 4 threads take a row, so that a workgroup has
// 1024 / D rows and no barrier, and the slots of a row are folded in order.
// With a workgroup per row the launch is bound by starting workgroups: 32
// layers of 8 heads, 128 rows a head, 54 us; 27 us here.  With few rows the
// many slots of one are better dealt to the workgroup.
template <int D>
__global__ __launch_bounds__(kCombThreads) void decode_combine_rows_kernel(
    Geo g, int64_t U, DecodeChunks ck, int32_t tq, int32_t mp, const int64_t* __restrict__ poff,
    const float* __restrict__ part_o,
    const float2* __restrict__ part_ml, float* __restrict__ out, float* __restrict__ lse) {
  constexpr int C4 = D / 4;
  constexpr int RW = kCombThreads / C4;
  const int64_t u = blockIdx.x;
  const int row = blockIdx.y * RW + threadIdx.x / C4;
  const int c4 = threadIdx.x % C4;
  const int len = (int)(poff[u + 1] - poff[u]);
  const DecCut cut = dec_cut(ck, (uint32_t)(poff[U] - poff[0]), U);
  const uint32_t at_row = (uint32_t)(poff[u] - poff[0]), s0 = at_row / cut.keys;
  const int nv = (int)dec_partials(cut, at_row, s0, (uint32_t)min(ck.cover, (int64_t)len));
  const int64_t base = (int64_t)dec_place(cut, at_row, s0, (uint32_t)u) * mp + row;  // + slot * mp
  if (len > ck.cover && blockIdx.y == 0 && threadIdx.x == 0) report_range(g);
  if (row >= tq * g.G) return;
  float m = -INFINITY, L = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  constexpr int Q = 4;  // slots in flight; those past the last are read again and not folded
  for (int i0 = 0; i0 < nv; i0 += Q) {
    float2 ml[Q];
    float4 o[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int64_t pr = base + (int64_t)min(i0 + i, nv - 1) * mp;
      ml[i] = part_ml[pr];
      o[i] = reinterpret_cast<const float4*>(part_o + pr * D)[c4];
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      if (i0 + i >= nv || ml[i].x == -INFINITY) continue;
      const float mn = fmaxf(m, ml[i].x);
      const float a = __builtin_amdgcn_exp2f(m - mn);  // 0 while m is -inf
      const float w = __builtin_amdgcn_exp2f(ml[i].x - mn);
      m = mn;
      L = fmaf(L, a, ml[i].y * w);
      acc.x = fmaf(acc.x, a, o[i].x * w);
      acc.y = fmaf(acc.y, a, o[i].y * w);
      acc.z = fmaf(acc.z, a, o[i].z * w);
      acc.w = fmaf(acc.w, a, o[i].w * w);
    }
  }
  const int h = (int)(u % g.H);
  const int64_t lb = u / g.H;
  const int b = (int)(lb % g.B);
  const int l = (int)(lb / g.B);
  const int t = row / g.G, gq = row % g.G;
  const int64_t orow = ((int64_t)l * g.B * tq + (int64_t)b * tq + t) * (g.H * g.G) + h * g.G + gq;
  acc.x /= L;
  acc.y /= L;
  acc.z /= L;
  acc.w /= L;
  if (!(isfinite(acc.x) && isfinite(acc.y) && isfinite(acc.z) && isfinite(acc.w)))
    report_nonfinite(g);
  *reinterpret_cast<dec_f32x4_any*>(out + orow * D + 4 * c4) =
      (dec_f32x4_any){acc.x, acc.y, acc.z, acc.w};
  if (lse && c4 == 0) lse[orow] = (m + __builtin_amdgcn_logf(L)) * kDecLn2;
}

template <int D, int NQT>
static certkv_status launch_decode(const DecodeArgs& a, hipStream_t s) {
  const Geo& g = a.g;
  const int mp = NQT * 32;
  // as many workgroups as stay resident at once (the occupancy query is made
  // once per device and kernel instance)
  constexpr int NT = 64 * DecShape<D, NQT>::NW;
  static std::atomic<int> per_cu[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CERTKV_EHIP;
  int nb = per_cu[dev].load(std::memory_order_relaxed);
  if (nb == 0) {
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, decode_kernel<D, NQT>, NT, 0) !=
        hipSuccess)
      return CERTKV_EHIP;
    nb = nb > 0 ? nb : 1;
    per_cu[dev].store(nb, std::memory_order_relaxed);
  }
  const int cus = device_cus(dev);
  if (cus <= 0) return CERTKV_EHIP;
  const int64_t max_items = a.ck.most + a.U - 1;
  const int64_t want = (int64_t)cus * nb;
  const unsigned grid = (unsigned)(max_items < want ? max_items : want);
  const uint16_t* q = static_cast<const uint16_t*>(a.q.ptr);
  const uint16_t* kp = static_cast<const uint16_t*>(a.k_packed);
  const uint16_t* vp = static_cast<const uint16_t*>(a.v_packed);
  CERTKV_LAUNCH("decode", (decode_kernel<D, NQT>), dim3(grid), dim3(NT), 0, s, g, a.U, a.ck, a.tq,
                mp, q, a.q.s_layer, a.q.s_token, a.q.s_head, kp, vp, a.packed_offsets, a.part_o, a.part_ml);
  const int M = a.tq * g.G;
  constexpr int RW = 4 * kCombThreads / D;
#define CERTKV_COMBINE(CL)                                                                         \
  CERTKV_LAUNCH("decode_combine", (decode_combine_kernel<D, CL>), dim3((unsigned)a.U, (unsigned)M), \
                dim3(kCombThreads), 0, s, g, a.U, a.ck, a.tq, mp,                                   \
                a.packed_offsets, (const float*)a.part_o, (const float2*)a.part_ml, a.out, a.lse,  \
                a.cl, q, a.q.s_layer, a.q.s_token, a.q.s_head)
  if (a.cl.m > 0)
    CERTKV_COMBINE(true);
  else if (a.U * M < 8192)
    CERTKV_COMBINE(false);
  else
    CERTKV_LAUNCH("decode_combine", (decode_combine_rows_kernel<D>),
                  dim3((unsigned)a.U, (unsigned)((M + RW - 1) / RW)), dim3(kCombThreads), 0, s, g,
                  a.U, a.ck, a.tq, mp, a.packed_offsets,
                  (const float*)a.part_o, (const float2*)a.part_ml, a.out, a.lse);
#undef CERTKV_COMBINE
  return CERTKV_OK;
}

template <int D>
static certkv_status launch_decode_d(const DecodeArgs& a, hipStream_t s) {
  switch (decode_nqt(a.tq * a.g.G)) {
    case 1: return launch_decode<D, 1>(a, s);
    case 2: return launch_decode<D, 2>(a, s);
    case 4: return launch_decode<D, 4>(a, s);
    case 8: return launch_decode<D, 8>(a, s);
    default: return launch_decode<D, 16>(a, s);
  }
}

certkv_status run_decode(const DecodeArgs& a, hipStream_t s) {
  return a.g.D == 128 ? launch_decode_d<128>(a, s) : launch_decode_d<64>(a, s);
}

// Workgroups resident at once on the device the chunks are cut for: by LDS two
// per compute unit at 128 dims and four at 64, by registers three with four query
// tiles of 64 dims and one with eight and more.
static int decode_parts(int D, int nqt) {
  return 256 * (nqt >= 8 ? 1 : D == 128 ? 2 : nqt == 4 ? 3 : 4);
}

DecodeChunks decode_chunks(int D, int tq, int G, int64_t cover_rows, int64_t rows) {
  const int nqt = decode_nqt(tq * G);
  DecodeChunks c;
  c.cover = (cover_rows + 4095) / 4096 * 4096;
  c.keys_min = 128;
  c.parts = decode_parts(D, nqt);
  const int64_t shortest = (rows + c.keys_min - 1) / c.keys_min;
  c.most = c.parts < shortest ? c.parts : (int32_t)shortest;
  c.sums = (rows + (1 << kDecSumShift) - 1) >> kDecSumShift;
  return c;
}

int64_t decode_partials(const DecodeChunks& c, int64_t U) { return c.sums + c.most + U; }

}  // namespace certkv
