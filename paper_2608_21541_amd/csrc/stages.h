// Argument blocks and host launchers of the kernel stages (internal).
#pragma once

#include <vector>

#include "common.h"

namespace certkv {

struct ScoreArgs {
  Geo g;
  certkv_tensor q, k;
  int32_t dtype;
  float* scores;
  double* ksum;
  float2* part;
  float* lse2;
  float* kpart;
  int32_t* flag;  // [U] units whose shift-free row sums left the safe range
  const float* lse_in;  // optional caller row log-sum-exp [L][B*w][Hq]
  float* lse_out;       // optional row log-sum-exp out, same layout
  int32_t keys_per_block;   // pass 1 (and its partials)
  int32_t nkb_max;
  int32_t keys_per_block2;  // pass 2 (and its key-sum partials)
};
// Query tiles of 32 rows covering the M window rows, rounded up to a power of two.
inline int score_nqt(int M) {
  int t = 1;
  while (t * 32 < M) t *= 2;
  return t;
}
certkv_status run_score(const ScoreArgs& a, const SeqTab& st, int max_len, hipStream_t s);

constexpr int kSortRun = 4096;  // elements a workgroup sorts in LDS at most
constexpr int kSortOver = 32;   // samples per bucket
constexpr int kSortNb = kSortRun / kSortOver;  // buckets of a unit at most
// Buckets of a unit of n elements: one up to kSortRun, else of half of it on
// average (a bucket spans the gaps between 32 samples, so with keys in no
// particular order about 3 in a million exceed twice the average).
__host__ __device__ inline int sort_nb(int n) {
  return n <= kSortRun ? 1 : (int)((2 * (int64_t)n + kSortRun - 1) / kSortRun);
}
// Tiles of a unit of n elements.
__host__ __device__ inline int sort_tiles(int n) {
  return (int)(((int64_t)n + kSortRun - 1) / kSortRun);
}
struct SortArgs {
  Geo g;
  const float* scores;
  uint32_t *keysA, *keysB, *keys_out;
  int32_t *valsA, *valsB, *perm_out;
  double* ssum;
  // split by value into buckets (nb_max = buckets of the longest sequence; 1:
  // every unit fits one LDS sort; 0: one workgroup sorts a unit through memory)
  int32_t nb_max;
  // one entry per bucket, or per tile of kSortRun elements, of the launch (part_base)
  uint64_t* splitters;       // per bucket
  uint2* windows;            // per bucket: keys that most of it lies between
  uint32_t* counts;          // per tile, [nb_max]
  uint32_t* bucket_start;    // per bucket
  double* tile_sum;          // per tile
};
certkv_status run_sort(const SortArgs& a, const SeqTab& st, hipStream_t s);

constexpr int kCurveChunk = 512;  // ranks a curves workgroup walks at a time
struct CurveArgs {
  Geo g;
  const uint32_t* sorted_keys;
  const int32_t* perm;
  const double* ssum;
  certkv_tensor v;
  int32_t dtype;
  float* curves;
  double* vsum;
  int32_t seg_chunks;        // chunks per segment, and segments of the longest
  int32_t nseg_max;          // sequence (1: one workgroup walks a whole unit)
  double* segtot;            // [U][nseg_max][32][d/32 + 2] segment totals
};
certkv_status run_curves(const CurveArgs& a, const SeqTab& st, hipStream_t s);

struct AllocArgs {
  Geo g;
  const float* curves;
  float* cmin;      // [U][nblk_max][2] minima of c over the two halves of each block
  float* cmaxb;     // [U][nblk_max] block maxima of c
  int32_t* cpos;    // [U][nblk_max] smallest position of the block minimum
  double* dmax;     // [U][nblk_max] block maxima of c(i+1) - c(i)
  int32_t nblk_max;
  int32_t steps;
  int32_t* budgets;
  int64_t* repairs;
  int32_t* sync;    // alloc_sync_words() words: cross-workgroup bisection (optional)
  int32_t chunk_blocks;  // blocks per chunk of the hull filter: 2 or 8
  uint2* hull_pts;   // per chunk, [alloc_chunk_points()]: its hull points, then its unit's
  int32_t* hull_cnt; // per chunk (of the launch: part_base)
  int32_t* unit_cnt; // [U]
  float* unit_max;   // [U]
  int32_t* done;     // [L*B] set where the hull kernel allocated
};
size_t alloc_sync_words();
size_t alloc_chunk_points();
certkv_status run_allocate(const AllocArgs& a, const SeqTab& st, hipStream_t s);

// Units up to which the selection sums the offsets by itself: a launch of one
// workgroup takes 4.7 us, the sum in every workgroup 1 us (the pass 1.1 to 1.6 us shorter).
constexpr int kSelOwnOffsets = 1024;
struct SelectArgs {
  Geo g;
  bool own_offsets;          // kept_offsets and packed_offsets are written by the selection
  const float* scores;
  const uint32_t* sorted_keys;
  const int32_t* perm;
  int32_t* budgets;
  int64_t* kept_offsets;
  int64_t* packed_offsets;
  int32_t* kept_idx;
  int64_t capacity;
  double* evicted_sum;
  double* total_sum;
  uint64_t* bitmap;
  int32_t bm_stride;
  uint8_t* mask;             // optional [L][H][T]: 1 at kept positions, else 0
};
certkv_status run_coverage(const Geo& g, const SeqTab& st, const float* scores,
                           const uint32_t* sorted_keys, double retain, int32_t* budgets,
                           hipStream_t s);
certkv_status run_clamp(const Geo& g, const SeqTab& st, int32_t* budgets, hipStream_t s);
certkv_status run_offsets(int64_t U, int32_t slot, const int32_t* budgets, int64_t* kept_offsets,
                          int64_t* packed_offsets, hipStream_t s);
certkv_status run_uniform_budgets(const Geo& g, const SeqTab& st, int32_t* budgets, hipStream_t s);
certkv_status run_select(const SelectArgs& a, const SeqTab& st, hipStream_t s);
struct TailArgs {
  Geo g;
  int32_t dtype;
  const float* scores;
  certkv_tensor k, v;
  const int64_t* kept_offsets;
  const int32_t* kept_idx;
  uint64_t* bitmap;
  int32_t bm_stride;
  int32_t nsplit;            // gather workgroups per unit
  int32_t nslice;            // mass workgroups per unit (standalone path)
  double* kpart;             // [U][nsplit][2][D] partial kept sums
  double* mpart;             // [U][nslice][3] partial masses (standalone path)
  const double* evicted_sum; // [U] from the selection pass, or NULL
  const double* total_sum;   // [U] from the selection pass, or NULL
  const double* ksum;
  const double* vsum;
  float* k_star;
  float* v_star;
  double* tail_mass;
  void* k_packed;
  void* v_packed;
  int32_t* pos_packed;
  bool do_tail, do_compact;
};
certkv_status run_bitmap(const TailArgs& a, const SeqTab& st, int64_t words_total, bool clear,
                         hipStream_t s);
certkv_status run_tail(const TailArgs& a, const SeqTab& st, hipStream_t s);
size_t score_smem_bytes(const Geo& g, int32_t dtype);

struct ClusterArgs {
  Geo g;
  int32_t dtype;
  int32_t m;                    // groups per head
  const int32_t* perm;          // [L][H][T] rank order of the pass
  const int32_t* budgets;       // [U]
  certkv_tensor k, v;
  void* kbar;                   // [U][m][d] in the cache dtype
  void* vbar;
  int32_t* count;               // [U][m]
  float* rk;                    // [U][m] key radii
  float* rv;                    // [U][m] value radii
  float* vmax_kept;             // [U]
};
certkv_status run_clusters(const ClusterArgs& a, const SeqTab& st, hipStream_t s);
certkv_status run_clusters_clear(float* vmax_kept, int64_t U, hipStream_t s);  // before run_clusters

// Optional clustered-tail terms of a decode (added in the combine).
struct DecodeClusters {
  int32_t m;                    // 0: none
  const uint16_t* kbar;         // [U][m][d] bf16
  const uint16_t* vbar;
  const int32_t* count;
  const float* rk;
  const float* rv;
  const float* vmax_kept;
  float* bound;                 // optional [L][B*tq][Hq] certificate (inf if it does not hold)
};

// How the packed rows are cut into chunks (see decode.hip).
struct DecodeChunks {
  int64_t cover;                // rows of a segment that are attended
  int32_t most;                 // chunks the workspace has room for
  int64_t sums;                 // and partials of a single segment of all the rows
  int32_t keys_min;             // shortest chunk
  int32_t parts;                // workgroups resident at once
};

struct DecodeArgs {
  Geo g;
  int64_t U;
  int32_t tq;                   // new queries per sequence
  DecodeChunks ck;
  certkv_tensor q;              // [L][B*tq][Hq][d] bf16
  const void* k_packed;         // [P][d] bf16
  const void* v_packed;
  const int64_t* packed_offsets;
  float* part_o;                // [decode_partials()][mp][d]
  float2* part_ml;              // [decode_partials()][mp]
  float* out;                   // [L][B*tq][Hq][d]
  float* lse;                   // optional [L][B*tq][Hq]
  DecodeClusters cl;
};
// Query tiles of 32 rows for M decode rows, rounded up to a power of two.
inline int decode_nqt(int M) {
  int t = 1;
  while (t * 32 < M) t *= 2;
  return t;
}
certkv_status run_decode(const DecodeArgs& a, hipStream_t s);
// rows: of all segments together, at most; cover_rows: of one.
DecodeChunks decode_chunks(int D, int tq, int G, int64_t cover_rows, int64_t rows);
int64_t decode_partials(const DecodeChunks& c, int64_t U);  // partials of a call at most

certkv_status run_packed_from_kept(int64_t U, int32_t slot, const int64_t* kept_offsets,
                                   int64_t* packed_offsets, hipStream_t s);
}  // namespace certkv
