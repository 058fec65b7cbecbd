// Exact k nearest neighbours on gfx950 as a filtered matrix product.
//
// Order: squared Euclidean distance in FP32 (sum_k (q_k - x_k)^2, features in
// order), ties to the lower index, the query itself excluded.
//
// Every coordinate, less the centre of its feature and scaled by a power of two,
// is split into hi = fp16(x) and lo = fp16(x - hi) (22 significant bits together).
// The matrix cores compute the ranking value
//     a(q, c) = q.c - |c|^2 / 2          (the distance is |q|^2 - 2 a)
// with FP32 accumulation, from one of
//     1 segment    hi.hi
//     3 segments   hi.lo + lo.hi + hi.hi  (close to FP32 accuracy)
// and each query keeps its KP best candidates by a.  These are ranked by their exact
// FP32 distances, and the answer is certified: with E a bound on the error of a
// (Cauchy-Schwarz on the rows' actual rounding residuals, plus the worst case of the
// accumulation), a candidate that was dropped has a <= a_last + E, hence a distance
// of at least |q|^2 - 2 (a_last + E); the answer stands when its k-th distance lies
// below that.  E is taken over the candidates that can be an answer at all, those of
// norms up to |q| and the k-th distance, so that rows far off spoil none but their
// own.  What is not certified goes through a band (see there): tiles of like queries
// with centres of their own, the exact distances of all candidates whose value may
// be an answer's, with one segment, then with three, and over all candidates in the
// end.  So the answers are those of the order above whatever the data; what depends
// on the data is the time, here for 400,000 x 100 points, k = 2: 53 ms (a mixture of
// clusters, distances a quarter of their offsets, with or without a coordinate far
// off), 156 (standardised binary features, 4,096 different rows), 193 (clusters with
// distances 1/60 of the offsets), 210 (equal points), 373 (1/3000).  The search before
// the filter, three segments for every pair and no certificate, took 149 to 247.
// Few candidates or queries go to their exact distances at once (direct_pays).
//
// knn_filter_kernel: a block of 8 waves owns 256 queries and a range of candidate
// tiles of 256; wave (wc, wq) computes 128 candidates x 64 queries with
// v_mfma_f32_32x32x16_f16 (candidates on the rows, so a lane's 64 values of a query
// column stay in its registers).  Operands are laid out by the split kernel as the
// LDS stage images themselves: 256 rows x 32 features = 16 KB, in slot order, so a
// stage is filled by global_load_lds_dwordx4 from consecutive addresses, without
// bounds checks (rows past the end are zero, their start value -3e38).  The values
// never leave the registers: a lane compares the maximum of 16 of them with its
// query's threshold (the KP-th best so far), and only hits go to the query's list in
// LDS, which is cut to its KP best when it fills up.  A sweep starts with a short run
// over its first tiles that only tracks the maxima of 32 groups of candidates per
// query: at least KP candidates reach the KP-th largest of them, so the lists never
// see the flood of a cold start.  After it a query has about KP ln(M / 4096) hits in
// a sweep, in whatever order the rows come: the candidates are swept in one of their
// own (knn_order_kernel).
// What bounds it: the matrix cores, at the clock that the power limit leaves
// them (1.7 GHz instead of 2.4 in these loops): per K step of 32 a CU spends
// 1,024 cycles in MFMAs, beside 768 of operand reads and 256 of stage writes.
// Measured (whole call, exact graph): 400,000 x 100, k = 2 149.6 -> 53 ms (the sweep
// 49 ms, 45 of them without any hit: 0.83 PFLOP/s of products); 70,000 x 784, k = 5
// 52.4 -> 14.9 ms; 48,600 x 128, k = 20 24.8 -> 4.6 ms.  Before, three segments
// always, each score through LDS to two threads per query row with a register list.
// Waves of 64 x 64 (16 per block), a ring of three stages and per-register ballots
// measured the same or slower: what a hit costs (about 0.2 us of its wave) is what is
// left above the products.
#include <cfloat>
#include <cmath>
#include <cstring>
#include <numeric>
#include <type_traits>

#include "knn_internal.h"
#include "knn_rank.h"

namespace ivhd {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int FT = 256;                  // rows per tile (queries and candidates)
constexpr int FK = 32;                   // features per stage
constexpr int kTileHalves = FT * FK;     // one operand's share of a stage (16 KB)
constexpr int kFilterWaves = 8;
constexpr int kCandWaves = kFilterWaves / 4;   // waves along the candidates of a tile
constexpr int NI = FT / kCandWaves / 32;       // 32 x 32 blocks of a wave along the candidates
constexpr int kFilterThreads = 64 * kFilterWaves;
constexpr int64_t kCus = 256;
constexpr int kRing = 2;                 // stages in LDS: the loads of one fly while the other is used
constexpr int kListPlaces = 44;          // places of a query's list (LDS: 64 KB ring + 88 KB lists)
constexpr float kNoValue = -2.9e38f;     // threshold of a list that is not full
constexpr float kPadStart = -3.0e38f;    // start value of rows past the end (below kNoValue)

// slot of 16-byte chunk `chunk` (8 features) of row `row` in a stage image:
// an operand read touches rows r..r+31 at chunk c (lanes 0-31) and c + 1
// (lanes 32-63); any eight consecutive rows at one chunk, and any four at
// both, fall on distinct 16-byte bank groups
__device__ __forceinline__ int tile_slot(int row, int chunk) {
  return row * 4 + (chunk ^ ((row & 2) | ((row >> 2) & 1)));
}

// A candidate of a list: the value's bits made monotone above, the
// complement of its id below, so that a larger key is a better candidate
// (larger a, then lower id).  0: none.
__device__ __forceinline__ uint64_t cand_key(float a, int32_t id) {
  const uint32_t u = __float_as_uint(a);
  return (uint64_t)(u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u)) << 32 | (uint32_t)~id;
}
__device__ __forceinline__ int32_t key_id(uint64_t k) { return (int32_t)~(uint32_t)k; }
__device__ __forceinline__ float key_value(uint64_t k) {
  const uint32_t u = (uint32_t)(k >> 32);
  return __uint_as_float(u ^ (~(uint32_t)((int32_t)u >> 31) | 0x80000000u));
}

// ---- operands ---------------------------------------------------------------

// Centre and spread of a set of rows, from kSampleRows of them spread over it:
// mean[n] the median of the sample's feature n, spread the largest over the
// features of a quantile of |x - mean| (float bits; zero before use): the third
// quartile, or what only three of the sample exceed where that is 0.  Centred data
// have smaller norms, hence smaller error bounds; median and quantile, since rows
// far off (a missing-value code) would pull a mean away from all the others and
// push those below the FP16 grid; and a value of the data as the centre, so that
// differences from it stay on the data's own grid.
constexpr int kSampleRows = 255;

__global__ void __launch_bounds__(256) knn_sample_kernel(const float *__restrict__ X, int64_t M, int N,
                                                         float *__restrict__ mean, uint32_t *__restrict__ spread) {
  __shared__ __attribute__((aligned(16))) uint32_t v[256];
  __shared__ float quartile, most;
  const int n = blockIdx.x, p = threadIdx.x;
  const int rows = M < kSampleRows ? (int)M : kSampleRows;
  const bool on = p < rows;
  // place of the thread's value among the sample's: by the top 24 bits of its
  // order, then by row (256 comparisons, of keys that differ)
  auto rank_of = [&](float x) {
    const uint32_t u = __float_as_uint(x);
    const uint32_t key = on ? ((u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u)) & ~255u) | (uint32_t)p : ~0u;
    v[p] = key;
    __syncthreads();
    int rank = 0;
#pragma unroll 8
    for (int e = 0; e < 256; e += 4) {
      const u32x4 w = *reinterpret_cast<const u32x4 *>(v + e);
#pragma unroll
      for (int u = 0; u < 4; ++u) rank += w[u] < key ? 1 : 0;
    }
    __syncthreads();
    return on ? rank : -1;
  };
  const float x = on ? X[(int64_t)p * M / rows * N + n] : 0.f;
  if (rank_of(x) == rows / 2) mean[n] = most = x;
  __syncthreads();
  const float far = fabsf(x - most);
  const int rank = rank_of(far);   // (every thread has read most)
  if (rank == rows * 3 / 4) quartile = far;
  if (rank == (rows > 4 ? rows - 4 : rows - 1)) most = far;
  __syncthreads();
  const float q = quartile > 0.f ? quartile : most;
  if (p == 0 && q > 0.f) atomicMax(spread, __float_as_uint(q));   // non-negative floats compare as integers
}

// The order in which candidates are swept: place p holds row p stride mod M, the
// stride about 0.618 M and prime to M, so that every stretch of places is spread
// evenly over the rows.  Rows as they come may lie along a path (a series in time),
// and then every candidate on the way to a query is nearer than all before it: each
// a hit (100,000 x 100 points along a line: 402 ms as they come).
__global__ void knn_order_kernel(int64_t M, int64_t stride, int32_t *__restrict__ order) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < M) order[p] = (int32_t)(p * stride % M);
}

// Class of a row by its squared norm: a factor of two to a class
__device__ __forceinline__ int norm_class(float norm2) {
  return (int)(__float_as_uint(norm2) >> 23 & (kNormClasses - 1));   // (a NaN's sign aside)
}

__device__ __forceinline__ float clamp_half(float t) { return fminf(fmaxf(t, -65504.f), 65504.f); }

// Stage images of scale * (X - mean) (rows taken through `map` when given, -1: a
// row of zeros; mean_stride > 0: a centre for each tile), and in those units the rows' squared norms and rounding residuals, start values and
// the statistics of the set.  A coordinate beyond the FP16 range is held at its
// end: all of it that is missing counts as the row's residual.
// 16 lanes per row, 8 features per lane and step; a block walks rows 16 at a
// time so that the maxima cost a block one atomic each.
__global__ void __launch_bounds__(256) knn_split_kernel(const float *__restrict__ X, int64_t M, int N, int nk,
                                                        const int32_t *__restrict__ map,
                                                        const float *__restrict__ means, int64_t mean_stride,
                                                        float scale, _Float16 *__restrict__ hi,
                                                        _Float16 *__restrict__ lo, float *__restrict__ norms,
                                                        float *__restrict__ res,
                                                        float *__restrict__ start, KnnStats *__restrict__ stats,
                                                        bool vec) {
  __shared__ float smax[4];
  __shared__ uint32_t cls[kNormClasses];
  const int g = threadIdx.x & 15;
  const int64_t rows = (M + FT - 1) / FT * FT;
  float top_s = 0.f;
  if (stats) cls[threadIdx.x] = 0;
  __syncthreads();
  for (int64_t row = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4); row < rows; row += (int64_t)gridDim.x * 16) {
    const int64_t src = row < M ? (map ? (int64_t)map[row] : row) : -1;
    const bool real = src >= 0;
    const float *x = X + (real ? src : 0) * N, *mean = means + row / FT * mean_stride;
    const int64_t base = row / FT * nk * kTileHalves;
    const int r = (int)(row % FT);
    float s = 0.f, e = 0.f;
    for (int c = g; c < nk * 4; c += 16) {
      float v[8];
      if (vec && 8 * c + 8 <= N) {
        const floatx4 u = *reinterpret_cast<const floatx4 *>(x + 8 * c) - *reinterpret_cast<const floatx4 *>(mean + 8 * c);
        const floatx4 w =
            *reinterpret_cast<const floatx4 *>(x + 8 * c + 4) - *reinterpret_cast<const floatx4 *>(mean + 8 * c + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          v[j] = real ? u[j] : 0.f;
          v[j + 4] = real ? w[j] : 0.f;
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = real && 8 * c + j < N ? x[8 * c + j] - mean[8 * c + j] : 0.f;
      }
      halfx8 h, l;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float t = v[j] * scale;
        s += t * t;
        h[j] = (_Float16)clamp_half(t);
        const float d = t - (float)h[j], dc = clamp_half(d);
        e += d == dc ? d * d : INFINITY;   // (what the low part cannot hold either)
        l[j] = (_Float16)dc;
      }
      const int64_t at = base + (int64_t)(c >> 2) * kTileHalves + tile_slot(r, c & 3) * 8;
      if (hi) *reinterpret_cast<halfx8 *>(hi + at) = h;
      if (lo) *reinterpret_cast<halfx8 *>(lo + at) = l;
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
      s += __shfl_xor(s, o, 64);
      e += __shfl_xor(e, o, 64);
    }
    if (g == 0) {
      if (norms && row < M) norms[row] = s;
      if (res && row < M) res[row] = e;
      if (start) start[row] = real ? -0.5f * s : kPadStart;
      if (stats && e > 0.f) atomicMax(&cls[norm_class(s)], __float_as_uint(e));
    }
    top_s = fmaxf(top_s, s);
  }
  if (!stats) return;
#pragma unroll
  for (int o = 32; o >= 16; o >>= 1) top_s = fmaxf(top_s, __shfl_xor(top_s, o, 64));
  if ((threadIdx.x & 63) == 0) smax[threadIdx.x >> 6] = top_s;
  __syncthreads();
  if (threadIdx.x == 0)   // non-negative floats compare as integers
    atomicMax(&stats->norm2, __float_as_uint(fmaxf(fmaxf(smax[0], smax[1]), fmaxf(smax[2], smax[3]))));
  if (cls[threadIdx.x]) atomicMax(&stats->res[threadIdx.x], cls[threadIdx.x]);
}

constexpr double kUp = 1.0 + 1e-6, kU23 = 1.1920928955078125e-7;

// relative error of an FP32 sum of N squares: 16 lanes, then a tree
__host__ __device__ __forceinline__ double sum_error(int N) { return (N / 16 + 16) * kU23; }

// res[c] <- the largest of classes 0..c, as a residual and not its square, rounded up
__global__ void __launch_bounds__(kNormClasses) knn_classes_kernel(KnnStats *stats, int N) {
  __shared__ uint32_t m[kNormClasses];
  const int t = threadIdx.x;
  m[t] = stats->res[t];
  for (int o = 1; o < kNormClasses; o *= 2) {
    __syncthreads();
    const uint32_t w = t >= o ? m[t - o] : 0u;
    __syncthreads();
    m[t] = w > m[t] ? w : m[t];
  }
  stats->res[t] = __float_as_uint((float)(sqrt((double)__uint_as_float(m[t]) * (1 + sum_error(N))) * (kUp * kUp)));
}

// ---- the filter -------------------------------------------------------------

struct FilterArgs {
  const _Float16 *Qh, *Ql, *Ch, *Cl;   // stage images; the lo ones only with three segments
  const float *start;                  // [tiles * FT]
  int nk;                              // stages per segment
  int64_t nq;
  int64_t qb0, qb_step;                // query tile of item row r: qb0 + r qb_step
  int64_t nqb;                         // query tiles of this launch
  int splits;                          // candidate ranges
  int64_t tiles, tiles_per_split;
  int lead;                            // tiles that set the starting thresholds
  int64_t M, place_of;                 // row r is candidate r place_of mod M
  int self_mode;                       // 0 none, 1 the query's own row, 2 self[]
  const int32_t *self, *map;           // map: original row of query q (NULL: q)
  uint64_t *part;                      // [launch query][splits][KP]
  // band: hits of launch query t, those with values from limits[q] up; a query
  // tile of the launch has its own start values
  int64_t start_pitch;
  const float *limits;                 // by query (INFINITY or -INFINITY: no hits)
  int32_t *count, *ids;                // [t], [t][cap]; count goes on past cap
  int cap;
};

// block barrier that waits for this wave's LDS operations only: the stage
// loads in flight stay in flight
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// LDS writes as single instructions: the compiler would wait for every stage
// load in flight before each of them, since those write LDS too
__device__ __forceinline__ uint32_t lds_at(const void *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}
__device__ __forceinline__ void lds_put(uint64_t *p, uint64_t v) {
  asm volatile("ds_write_b64 %0, %1" ::"v"(lds_at(p)), "v"(v) : "memory");
}
template <typename T>
__device__ __forceinline__ void lds_put(T *p, T v) {
  static_assert(sizeof(T) == 4, "one dword");
  asm volatile("ds_write_b32 %0, %1" ::"v"(lds_at(p)), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_put2(uint64_t *p, uint32_t lo, uint32_t hi) {
  asm volatile("ds_write2_b32 %0, %1, %2 offset0:0 offset1:1" ::"v"(lds_at(p)), "v"(lo), "v"(hi) : "memory");
}
__device__ __forceinline__ void lds_max(float *p, float v) {
  asm volatile("ds_max_f32 %0, %1" ::"v"(lds_at(p)), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_put(uint8_t *p, uint32_t v) {
  asm volatile("ds_write_b8 %0, %1" ::"v"(lds_at(p)), "v"(v) : "memory");
}

// A query's list: KP places for its best so far (sorted once cut), then one
// area of (C - KP) / kOwners places for each of the lanes that hold its
// values: two lane halves x the waves along the candidates.  A lane appends to
// its own area without asking anybody; empty places hold 0.
constexpr int kOwners = 2 * kCandWaves;

// The list cut to its KP best, in place and sorted, the areas emptied; one
// lane per place.
template <int KP, int C>
__device__ __forceinline__ void cut_list(uint64_t *list, uint8_t *cnt, float *thr, int32_t *thr_id, int lane) {
  constexpr int AREA = (C - KP) / kOwners;
  uint64_t mine = 0;
  if (lane < C) {
    const int o = lane - KP;
    if (o < 0) {
      mine = list[lane];
    } else if (o % AREA < (int)cnt[o / AREA]) {   // as appended: id below, value above
      const uint64_t e = list[lane];
      mine = cand_key(__uint_as_float((uint32_t)(e >> 32)), (int32_t)(uint32_t)e);
    }
    lds_put(list + lane, mine);   // what is not counted is 0 from here on
  }
  int rank = 0;
#pragma unroll 11
  for (int j = 0; j < C; j += 2) {
    const uint64_t o0 = list[j], o1 = list[j + 1];
    rank += (o0 > mine ? 1 : 0) + (o1 > mine ? 1 : 0);
  }
  // the first KP places: the KP best, 0 where there are fewer
  if (lane < KP) lds_put(list + lane, (uint64_t)0);
  if (mine && rank < KP) lds_put(list + rank, mine);
  if (mine && rank == KP - 1) {
    lds_put(thr, key_value(mine));
    lds_put(thr_id, key_id(mine));
  }
  if (lane < kOwners) lds_put(cnt + lane, 0u);
}

// cuts the lists of the set bits, list q0 + bit each
template <int KP, int C>
__device__ __forceinline__ void cut_lists(uint32_t todo, int q0, uint64_t *lists, uint8_t *cnt, float *thr,
                                          int32_t *thr_id, int lane) {
  while (todo) {
    const int q = q0 + __builtin_ctz(todo);
    todo &= todo - 1;
    cut_list<KP, C>(lists + q * C, cnt + q * kOwners, thr + q, thr_id + q, lane);
  }
}

// KP: length of the lists.  SEG3: three segments, the small ones first, so that
// only the last one's additions round at the size of the value.  BAND: no lists;
// every value from the query's limit up is a hit.
template <int KP, bool SEG3, bool BAND>
__global__ void __launch_bounds__(kFilterThreads, kFilterWaves / 4) knn_filter_kernel(FilterArgs A) {
  constexpr int C = kListPlaces, RING = kRing, SEGS = SEG3 ? 3 : 1;
  constexpr int AREA = (C - KP) / kOwners;
  static_assert(C <= 64 && (C - KP) % kOwners == 0 && C % 2 == 0 && KP <= 32, "list shape");
  constexpr int kTrigger = AREA - (AREA > 4 ? 2 : 1);   // an area this full has the lists cut
  constexpr int SUB = 32 / (NI * kOwners);   // candidate groups per 32 x 32 block and lane: 32 per query
  // separate LDS objects: the compiler then knows that the lists are not what
  // the stage loads write, and does not wait for those at every list access
  __shared__ __attribute__((aligned(16))) _Float16 ring[RING * 2 * kTileHalves];   // [candidates 16 KB | queries 16 KB]
  __shared__ __attribute__((aligned(16))) float sStart[3 * FT];
  __shared__ __attribute__((aligned(16))) uint64_t sList[FT * C];
  __shared__ uint8_t sCnt[FT * kOwners];
  __shared__ float sThr[FT];
  __shared__ int32_t sThrId[FT];
  __shared__ int32_t sSelf[FT];
  __shared__ int32_t sFlag[2];           // [0] offer after which lists are to be cut, [1] one that left values over

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wc = 32 * NI * (wave >> 2), wq = 64 * (wave & 3);
  // XCD-aware items: blocks go to XCD b % 8; each XCD gets a contiguous run
  // of items, ordered by groups of four query tiles, then candidate range,
  // then query tile, so the blocks that run together on one L2 share query
  // panels and candidate tiles
  int64_t item;
  {
    const int64_t nb = gridDim.x, b = blockIdx.x, q = nb / kXcds, rem = nb % kXcds, x = b % kXcds, i = b / kXcds;
    item = x < rem ? x * (q + 1) + i : rem * (q + 1) + (x - rem) * q + i;
  }
  const int64_t full = A.nqb / 4 * 4 * A.splits;
  const int64_t gw = item < full ? 4 : A.nqb % 4, in_group = item < full ? item % (4 * A.splits) : item - full;
  const int64_t qrow = (item < full ? item / (4 * A.splits) * 4 : A.nqb / 4 * 4) + in_group % gw;
  const int split = (int)(in_group / gw);
  const int64_t qb = A.qb0 + qrow * A.qb_step;
  const int64_t q0 = qb * FT;
  const int t0 = (int)(split * A.tiles_per_split);
  const int t1 = (int)(t0 + A.tiles_per_split < A.tiles ? t0 + A.tiles_per_split : A.tiles);
  const int per_tile = A.nk * SEGS;
  // the tiles of this block in order: `lead` of them for the starting
  // thresholds, then all
  const int lead = !BAND && t1 > t0 ? min(A.lead, t1 - t0) : 0;
  const int ntiles = t1 > t0 ? lead + (t1 - t0) : 0;
  const int64_t nstages = (int64_t)ntiles * per_tile;

  // lead tiles: the maxima of 32 groups of candidates per query, each kept by
  // one lane, in the place of the lists (which are still empty)
  float *gm = reinterpret_cast<float *>(sList);
  constexpr int GP = FT + 1;   // pitch of a group's values

  if (tid < FT) {
    const int64_t q = q0 + tid;
    const int64_t orig = q < A.nq ? (A.map ? (int64_t)A.map[q] : q) : -1;
    // padding queries, and those without a limit, keep nothing
    sThr[tid] = q < A.nq ? (BAND ? (A.limits[q] > -INFINITY ? A.limits[q] : INFINITY) : kNoValue) : INFINITY;
    if (!BAND) sThrId[tid] = INT32_MAX;
    const int64_t own = orig < 0 ? -1 : (A.self_mode == 1 ? orig : (A.self_mode == 2 ? (int64_t)A.self[orig] : -1));
    sSelf[tid] = own >= 0 && own < A.M ? (int32_t)(own * A.place_of % A.M) : -1;
  }
  if constexpr (!BAND) {
    if (tid < 2) sFlag[tid] = -1;
    for (int e = tid; e < FT * kOwners; e += kFilterThreads) sCnt[e] = 0;
    for (int e = tid; e < FT * C; e += kFilterThreads) sList[e] = 0;
  }
  __syncthreads();
  if (lead > 0)
    for (int e = tid; e < 32 * GP; e += kFilterThreads) gm[e] = kNoValue;

  const float *start = BAND ? A.start + qrow * A.start_pitch : A.start;
  // stage issue: counters of the next stage to load
  int i_seq = 0, i_seg = 0, i_k = 0, i_slot = 0, i_start = 0;
  const uint32_t load_at = tid * 16;
  auto issue = [&]() __attribute__((always_inline)) {
    const int64_t i_tile = i_seq < lead ? t0 + i_seq : t0 + i_seq - lead;
    const _Float16 *c = (SEG3 && i_seg == 0 ? A.Cl : A.Ch) + (i_tile * A.nk + i_k) * kTileHalves;
    const _Float16 *q = (SEG3 && i_seg == 1 ? A.Ql : A.Qh) + (qb * A.nk + i_k) * kTileHalves;
    _Float16 *dst = ring + i_slot * 2 * kTileHalves;
    if (i_seg == 0 && i_k == 0) {   // the tile's start values, ahead of its first stage
      if (wave == 0)
        __builtin_amdgcn_global_load_lds((const void *)(reinterpret_cast<const char *>(start + i_tile * FT) + load_at),
                                         (lds_void *)(sStart + i_start * FT), 16, 0, 0);
      i_start = i_start == 2 ? 0 : i_start + 1;
    }
    // 64 lanes x 16 bytes per wave, load and operand
    unsigned char *at = reinterpret_cast<unsigned char *>(dst) + wave * 1024;
#pragma unroll
    for (int u = 0; u < 16 / kFilterWaves; ++u) {
      __builtin_amdgcn_global_load_lds((const void *)(reinterpret_cast<const char *>(c) + load_at + u * kFilterThreads * 16),
                                       (lds_void *)(at + u * kFilterThreads * 16), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((const void *)(reinterpret_cast<const char *>(q) + load_at + u * kFilterThreads * 16),
                                       (lds_void *)(at + kTileHalves * 2 + u * kFilterThreads * 16), 16, 0, 0);
    }
    i_slot = i_slot == RING - 1 ? 0 : i_slot + 1;
    if (++i_k == A.nk) {
      i_k = 0;
      if (++i_seg == SEGS) {
        i_seg = 0;
        ++i_seq;
      }
    }
  };

  __syncthreads();   // lists ready
  const int row = lane & 31;
  const int ql[2] = {wq + row, wq + 32 + row};
  float thr[2] = {sThr[ql[0]], sThr[ql[1]]};
  const int owner = 2 * (wave >> 2) + (lane >> 5);
  const int32_t self[2] = {sSelf[ql[0]], sSelf[ql[1]]};   // -1: none
  int mine[2] = {0, 0};   // entries in this lane's areas
  int32_t thr_id[2] = {INT32_MAX, INT32_MAX};
  // byte offsets of this lane's operand chunks in a stage; those of the
  // second 16 features are 32 bytes off (bit 1 of the chunk)
  const int at_c = tile_slot(wc + row, lane >> 5) * 16;
  const int at_q = kTileHalves * 2 + tile_slot(wq + row, lane >> 5) * 16;
  floatx16 acc[NI][2];
  // A lane's operand fragments of 16 features are read half a stage ahead of
  // the MFMAs that use them, so that LDS reads and MFMAs overlap.  Stage
  // st + 1 is entered in the middle of stage st: when this wave's loads of it
  // have landed (all but those of the stage after) and its reads of stage st
  // are done.  After the barrier that holds for every wave, and the slot of
  // stage st takes the next loads.
  int64_t issued = 0, st = 0;
  int c_start = 0;
  uint32_t at = 0;   // byte offset of the current slot
  constexpr uint32_t kSlot = 2 * kTileHalves * 2;
  const unsigned char *ring8 = reinterpret_cast<const unsigned char *>(ring);
  halfx8 a0[NI], b0[2], a1[NI], b1[2];
  auto read0 = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NI; ++i)   // 32 rows further: 32 * 4 slots of 16 bytes
      a0[i] = *reinterpret_cast<const halfx8 *>(ring8 + at + at_c + 2048 * i);
#pragma unroll
    for (int j = 0; j < 2; ++j) b0[j] = *reinterpret_cast<const halfx8 *>(ring8 + at + at_q + 2048 * j);
  };
  auto read1 = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NI; ++i) a1[i] = *reinterpret_cast<const halfx8 *>(ring8 + at + (at_c ^ 32) + 2048 * i);
#pragma unroll
    for (int j = 0; j < 2; ++j) b1[j] = *reinterpret_cast<const halfx8 *>(ring8 + at + (at_q ^ 32) + 2048 * j);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto mfma = [&](const halfx8 &a, const halfx8 &b, const floatx16 &c) __attribute__((always_inline)) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  };
  // The first MFMA of a half goes before the reads of the next: it is what
  // waits for its operands, and a wait after the reads would be for them too.
  auto finish_stage = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    at = at == (RING - 1) * kSlot ? 0 : at + kSlot;
    acc[0][0] = mfma(a1[0], b1[0], acc[0][0]);
    __builtin_amdgcn_sched_barrier(0);
    read0();   // (past the last stage: read, not used)
    __builtin_amdgcn_sched_barrier(0);
    acc[0][1] = mfma(a1[0], b1[1], acc[0][1]);
    if (issued < nstages) {
      issue();
      ++issued;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 1; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = mfma(a1[i], b1[j], acc[i][j]);
    __builtin_amdgcn_sched_barrier(0);
    ++st;
  };
  for (; issued < RING && issued < nstages; ++issued) issue();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  lds_barrier();
  read0();
  // the start values of a 32 x 32 block's rows
  auto starts = [&](int i) __attribute__((always_inline)) {
    const float *sv = sStart + c_start * FT + wc + 4 * (lane >> 5);
    floatx16 v;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const floatx4 w = *reinterpret_cast<const floatx4 *>(sv + 32 * i + 8 * g);
#pragma unroll
      for (int r = 0; r < 4; ++r) v[4 * g + r] = w[r];
    }
    return v;
  };
  for (int seq = 0; seq < ntiles; ++seq) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      floatx16 v = {};
      if (!SEG3) v = starts(i);
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = mfma(a0[i], b0[j], v);
    }
    read1();
    finish_stage();
#pragma unroll 1
    for (int ks = 1; ks < per_tile; ++ks) {
      if (SEG3 && ks == 2 * A.nk) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const floatx16 v = starts(i);
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] += v;
        }
      }
      acc[0][0] = mfma(a0[0], b0[0], acc[0][0]);
      __builtin_amdgcn_sched_barrier(0);
      read1();
      acc[0][1] = mfma(a0[0], b0[1], acc[0][1]);
#pragma unroll
      for (int i = 1; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma(a0[i], b0[j], acc[i][j]);
      finish_stage();
    }
    c_start = c_start == 2 ? 0 : c_start + 1;
    if constexpr (BAND) {
      // a lane's hits of the tile counted, then one atomic for their places; a
      // query that has too many is given up
      const int32_t c0 = (t0 + seq) * FT + wc + 4 * (lane >> 5);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        auto hits = [&](auto take) __attribute__((always_inline)) {
#pragma unroll
          for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              const floatx16 &v = acc[i][j];
              if (!__any(fmaxf(fmaxf(v[4 * g], v[4 * g + 1]), fmaxf(v[4 * g + 2], v[4 * g + 3])) >= thr[j])) continue;
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const int32_t id = c0 + 32 * i + 8 * g + r;
                if (v[4 * g + r] >= thr[j] && id != self[j]) take(id);
              }
            }
        };
        int n = 0;
        hits([&](int32_t) { ++n; });
        if (!__any(n > 0)) continue;
        const int64_t t = qrow * FT + ql[j];
        int at = n > 0 ? atomicAdd(&A.count[t], n) : 0;
        if (n > 0 && at + n > A.cap) {
          thr[j] = INFINITY;
          n = 0;
        }
        int32_t *to = A.ids + t * A.cap;
        if (n > 0) hits([&](int32_t id) { to[at++] = id; });
      }
      continue;
    }
    if (seq < lead) {
      // a lead tile (a query's own row is not a candidate, so its tile is
      // left out)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const bool own = self[j] >= 0 && self[j] / FT == t0 + seq;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int u = 0; u < SUB; ++u) {
            float m = acc[i][j][u * (16 / SUB)];
#pragma unroll
            for (int r = 1; r < 16 / SUB; ++r) m = fmaxf(m, acc[i][j][u * (16 / SUB) + r]);
            if (!own) lds_max(&gm[(owner * (NI * SUB) + i * SUB + u) * GP + ql[j]], m);
          }
      }
      if (seq == lead - 1) {
        // all candidates of their own: at least KP candidates reach the
        // KP-th largest of a query's 32 maxima
        lds_barrier();
        for (int p = 0; p < FT / kFilterWaves; p += 2) {
          const int q = wave * (FT / kFilterWaves) + p + (lane >> 5);
          const float m = gm[row * GP + q];
          int rank = 0;
#pragma unroll 8
          for (int e = 0; e < 32; ++e) {
            const float o = gm[e * GP + q];
            rank += o > m || (o == m && e < row) ? 1 : 0;
          }
          if (rank == KP - 1 && q0 + q < A.nq) lds_put(&sThr[q], m);
        }
        lds_barrier();
        for (int e = tid; e < GP * 16; e += kFilterThreads) lds_put(&sList[e], (uint64_t)0);
        lds_barrier();
        thr[0] = sThr[ql[0]];
        thr[1] = sThr[ql[1]];
      }
      continue;
    }
    // The values of a tile: D[i][j] of a 32 x 32 block sits in lane
    // j + 32 ((i / 4) % 2), register 4 (i / 8) + i % 4.  Values that beat the
    // threshold go to this lane's area of the query's list.  When an area is
    // full the tile is offered again once the lists have been cut; a lane's
    // ids ascend, so it then goes on after the last id that got in, and every
    // offer of a lane with values left gets at least one in: its area was cut
    // empty in between (a full area is one to be cut).
    int c0 = (t0 + seq - lead) * FT + wc + 4 * (lane >> 5);
    int32_t last[2] = {-1, -1};   // ids up to here have been dealt with
    for (int tries = 0; tries <= 16 * NI; ++tries) {   // a lane has 16 NI values per query
      asm volatile("" : "+v"(c0));   // keeps what derives from it out of the registers
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        uint64_t *area = &sList[ql[j] * C + KP + owner * AREA];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          float q[4];   // maxima of the registers by fours
#pragma unroll
          for (int g = 0; g < 4; ++g)
            q[g] = fmaxf(fmaxf(fmaxf(acc[i][j][4 * g], acc[i][j][4 * g + 1]), acc[i][j][4 * g + 2]),
                         acc[i][j][4 * g + 3]);
          if (!__any(fmaxf(fmaxf(fmaxf(q[0], q[1]), q[2]), q[3]) >= thr[j])) continue;
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            if (!__any(q[g] >= thr[j])) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float v = acc[i][j][4 * g + r];
              if (!__any(v >= thr[j])) continue;
              const int32_t id = c0 + 32 * i + 8 * g + r;
              if ((v > thr[j]) | ((v == thr[j]) & (id < thr_id[j])) && id != self[j] && id > last[j]) {
                if (mine[j] < AREA) {
                  lds_put2(area + mine[j], (uint32_t)id, __float_as_uint(v));
                  last[j] = id;
                }
                ++mine[j];
              }
            }
          }
        }
        lds_put(&sCnt[ql[j] * kOwners + owner], (uint32_t)min(mine[j], AREA));
      }
      const int most = max(mine[0], mine[1]);
      if (most >= kTrigger) lds_put(&sFlag[0], seq);
      if (most > AREA) lds_put(&sFlag[1], seq);
      lds_barrier();
      // Between the barriers below no wave sets a flag, so every wave sees
      // the same
      if (sFlag[0] != seq) break;
      const bool again = sFlag[1] == seq;
      // a round cuts every list with more than a few new entries, so that the
      // next round is far off
      constexpr int kLists = FT / kFilterWaves;   // of this wave
      int added = 0;
      if (lane < kLists)
#pragma unroll
        for (int o = 0; o < kOwners; ++o) added += sCnt[(wave * kLists + lane) * kOwners + o];
      cut_lists<KP, C>((uint32_t)__ballot(added > 2), wave * kLists, sList, sCnt, sThr, sThrId, lane);
      lds_barrier();   // flags read, thresholds written
      if (tid < 2) lds_put(&sFlag[tid], -1);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        thr[j] = sThr[ql[j]];
        thr_id[j] = sThrId[ql[j]];
        mine[j] = sCnt[ql[j] * kOwners + owner];
      }
      lds_barrier();   // flags reset
      if (!again) break;
    }
  }
  if constexpr (BAND) return;
  __syncthreads();
  static_assert(FT / kFilterWaves == 32, "a wave's lists in one mask");
  cut_lists<KP, C>(~0u, wave * 32, sList, sCnt, sThr, sThrId, lane);
  __syncthreads();
  for (int e = tid; e < FT * KP; e += kFilterThreads) {
    const int q = e / KP, p = e % KP;
    if (q0 + q < A.nq) A.part[((qrow * FT + q) * A.splits + split) * KP + p] = sList[q * C + p];
  }
}

// ---- survivors to answers -----------------------------------------------------

// an FP32 squared distance in scaled units (sc2: the scale's square), with its
// rounding and that of subnormal squares
__device__ __forceinline__ double scaled_above(float d, int N, double sc2) {
  return ((double)d * (1 + (N + 16) * kU23) + N * 1.5e-45) * sc2;
}

struct FinishArgs {
  const float *X, *Q;
  int N, nk, k, splits;
  int64_t nq, M;                 // queries of the call (compact ids), candidates
  int64_t qb0, qb_step, n_launch;   // launch query t is query (qb0 + t / FT qb_step) FT + t % FT
  const int32_t *map;            // original row of query q (NULL: q)
  const int32_t *order;          // row of candidate c
  int self_mode;                 // 0 none, 1 the query's own row, 2 self[]
  const int32_t *self;
  const uint64_t *part;
  int32_t *out_idx;
  float *out_dist;
  // certificate; norms and residuals in scaled units, centred
  const float *qnorm, *qres;     // [query] squared norm, squared residual
  const KnnStats *xs;            // of the candidates, after knn_classes_kernel
  double sub;                    // norm of the low parts' errors where they are subnormal
  float scale;
  int nseg;
  int32_t *fails;                // [0] count, then query ids
  float *fail_dist;              // of the fails: the k-th distance found
  int32_t *pilot;                // [3]: answers that lists of 8, 16, 32 would not certify (NULL: no pilot)
};

// The rows' own figures that bound the error of a query's values, in FP64 and
// rounded up by a factor well above its error
struct QueryBound {
  double nq, rq, nerr;   // norm, residual, relative error of an FP32 sum of N squares
};

// Bound on the error of a product of two rows of N features, of norms a and b
// and residuals ra and rb, computed in nseg segments from their images, where
// `sum` bounds the true partial sums together with the start value
__device__ __forceinline__ double product_error(int N, double sub, double a, double ra, double b, double rb, double sum,
                                                int nseg) {
  const double cross = a * rb + ra * (b + rb);   // the product less that of the high parts
  // one rounding to a feature, of no more than 2^-23 of the partial sum, all of
  // them one way (and a few for the operands' own)
  const double n = (double)N + 20;
  double err = n * kU23 * (sum + 2 * cross);
  if (nseg == 1) {
    err += kUp * cross;
  } else {
    // with hi + lo: the rounding of lo (2^-11 of the residual, or 2^-25 per
    // coordinate where lo is subnormal: sub), the product lo.lo, and the additions
    // that come before the large ones
    const double low = 1.5 * cross + (a + b) * sub;
    err += kUp * ((a + ra) * (rb / 2048 + sub) + (b + rb) * (ra / 2048 + sub) + ra * rb) + 3 * n * kU23 * low;
  }
  return err;
}

// the largest residual of a candidate of norm up to x
__device__ __forceinline__ double residual_at(const KnnStats *xs, double x, double nerr) {
  return __uint_as_float(xs->res[norm_class((float)(x * x * (1 + nerr) * kUp))]);
}

// Bound on the error of a against any candidate of norm up to x at a distance of
// up to dist (infinite when the rows' figures give none)
__device__ __forceinline__ double value_error(const FinishArgs &A, const QueryBound &B, double x, double dist) {
  // the largest partial sum: some of q.c's terms, those of |c|^2 and the rest of
  // no more than dist |c|, and the start value, of the other sign
  const double any = 0.5 * x * x + B.nq * x, close = x * x + dist * x;
  const double err = product_error(A.N, A.sub, B.nq, B.rq, x, residual_at(A.xs, x, B.nerr), close < any ? close : any,
                                   A.nseg) +
                     0.5 * B.nerr * x * x;   // and the start value's own
  return err == err ? err : INFINITY;
}

// KP lanes per query: merge the ranges' lists, exact FP32 distances of the
// survivors that can be among the k nearest, rank by (distance, id), certify.
template <int KP>
__global__ void __launch_bounds__(256) knn_finish_kernel(FinishArgs A) {
  __shared__ uint64_t sm[256];
  const int lane = threadIdx.x & 63, p = threadIdx.x & (KP - 1);
  const int g0 = lane & ~(KP - 1);   // first lane of the group
  uint64_t *grp = sm + (threadIdx.x & ~(KP - 1));
  const int64_t t = ((int64_t)blockIdx.x * 256 + threadIdx.x) / KP;
  const int64_t q = t < A.n_launch ? (A.qb0 + t / FT * A.qb_step) * FT + t % FT : A.nq;
  const bool on = q < A.nq;
  const uint64_t *src = A.part + t * A.splits * KP;
  uint64_t mine = on ? src[p] : 0;
  for (int s = 1; s < A.splits; ++s) {
    const uint64_t in = on ? src[s * KP + p] : 0;
    int rm = 0, ri = 0;
#pragma unroll 4
    for (int j = 0; j < KP; ++j) {
      const uint64_t m = __shfl(mine, g0 + j, 64), n = __shfl(in, g0 + j, 64);
      rm += (m > mine ? 1 : 0) + (n > mine ? 1 : 0);
      ri += (n > in ? 1 : 0) + (m > in ? 1 : 0);
    }
    grp[p] = 0;
    wave_fence();   // lanes write each other's places
    if (mine && rm < KP) grp[rm] = mine;
    if (in && ri < KP) grp[ri] = in;
    wave_fence();
    mine = grp[p];
    wave_fence();
  }
  const bool have = mine != 0;
  const int64_t orig = on ? (A.map ? (int64_t)A.map[q] : q) : 0;
  const double sc2 = (double)A.scale * A.scale;
  QueryBound B;
  B.nerr = sum_error(A.N);
  const double n2 = on ? (double)A.qnorm[q] : 0.0;
  B.nq = sqrt(n2 * (1 + B.nerr)) * kUp;
  B.rq = on ? sqrt((double)A.qres[q] * (1 + B.nerr)) * kUp : 0.0;
  int rank = 0, found = 0;
  uint64_t last = ~0ull, kth = 0;
#pragma unroll 4
  for (int j = 0; j < KP; ++j) {
    const uint64_t m = __shfl(mine, g0 + j, 64);
    rank += m > mine ? 1 : 0;
    found += m != 0 ? 1 : 0;
    last = m < last ? m : last;
  }
  uint64_t nth[3] = {0, 0, 0};   // the 8th, 16th and 32nd best
  for (int j = 0; j < KP; ++j) {
    const uint64_t m = __shfl(mine, g0 + j, 64);
    const int rj = __shfl(rank, g0 + j, 64);
    kth = rj == A.k - 1 && m ? m : kth;
#pragma unroll
    for (int l = 0; l < 3; ++l) nth[l] = rj == (8 << l) - 1 ? m : nth[l];
  }
  // A candidate whose norm exceeds the query's by more than the k-th distance is
  // farther than that, whatever its value: only norms up to `reach` matter, and a
  // row far from all others spoils no bound but its own.  The k best values bound
  // the k-th distance from above with the error that goes with the reach so far.
  bool near = have;   // may be among the k nearest
  double reach = sqrt((double)__uint_as_float(A.xs->norm2) * (1 + B.nerr)) * kUp;
  if (kth != 0) {
    double err = value_error(A, B, reach, INFINITY);
    for (int it = 0; it < 4 && reach > 2 * B.nq; ++it) {   // (not far off: little to gain)
      const double far2 = n2 * (1 + B.nerr) - 2.0 * ((double)key_value(kth) - err);
      const double far = sqrt(far2 > 0 ? far2 : 0.0) * kUp, r = (B.nq + far) * kUp;
      const bool less = r < 0.75 * reach;
      if (r < reach) reach = r;
      err = value_error(A, B, reach, far + 2 * kU23 * (B.nq + reach));
      if (!less) break;
    }
    // a value more than two errors below the k-th best cannot be (the slack
    // covers the rounding of the distances themselves)
    const double slack = (A.N + 16) * kU23 * (n2 + reach * reach);
    near = have && !((double)key_value(mine) < (double)key_value(kth) - 2.0 * err - slack);
  }
  float d = FLT_MAX;
  const int32_t id = near ? A.order[key_id(mine)] : INT32_MAX;
  if (near) d = exact_distance(A.Q + orig * A.N, A.X + (int64_t)id * A.N, A.N, rows_are_vec4(A.X, A.Q, A.N));
  rank = 0;
#pragma unroll 4
  for (int j = 0; j < KP; ++j) {
    const float dj = __shfl(d, g0 + j, 64);
    const int32_t ij = __shfl(id, g0 + j, 64);
    rank += (dj < d || (dj == d && (ij < id || (ij == id && j < p)))) ? 1 : 0;
  }
  if (on && rank < A.k) {
    A.out_idx[orig * A.k + rank] = near ? id : -1;
    if (A.out_dist) A.out_dist[orig * A.k + rank] = d;
  }
  if (on && rank == A.k - 1) {
    // The least squared distance of a candidate that is not among the first L of
    // the list, between the centred rows and (their rounding: 2^-24 of each
    // row) between the given ones, must lie above the k-th distance.
    const double top = scaled_above(d, A.N, sc2);
    const double r = (B.nq + sqrt(top)) * kUp, x = r < reach ? r : reach;
    const double shift = 0.5 * kU23 * (B.nq + x), dist = (sqrt(top) + shift) * kUp;
    const double err = value_error(A, B, x, dist);
    auto certified = [&](uint64_t last) {
      const double least = n2 * (1 - B.nerr) - 2.0 * ((double)key_value(last) + err);
      const double moved = sqrt(least > 0 ? least : 0.0) - shift;
      return top < (moved > 0 ? moved * moved : 0.0) * (1 - 1e-12);
    };
    // a list that is not full is the answer if it holds all there are
    auto complete = [&]() {
      const int64_t own = A.self_mode == 1 ? orig : (A.self_mode == 2 ? (int64_t)A.self[orig] : -1);
      return found >= A.M - (own >= 0 && own < A.M ? 1 : 0);
    };
    if (A.pilot) {
      for (int l = 0; l < 3; ++l) {
        const int len = 8 << l;
        if (len <= KP && (found < len ? !complete() : len < A.k || !certified(nth[l]))) atomicAdd(&A.pilot[l], 1);
      }
    } else if (found < KP ? !complete() : !certified(last)) {
      const int32_t at = atomicAdd(&A.fails[0], 1);
      A.fails[1 + at] = (int32_t)orig;
      A.fail_dist[at] = d;
    }
  }
}

// ---- answers from exact distances of many candidates ---------------------------

// best: a wavefront's 64 best keys (distance above, id below) sorted over its
// lanes, of which the first k count; the keys of a wavefront differ.  Of many that
// can be among them the least goes first, so that no more than k go in (along a
// line every key may be less than the one before it).
__device__ __forceinline__ void offer_sorted(uint64_t &best, uint64_t key, int lane, int k) {
  uint64_t mask = __ballot(key < __shfl(best, k - 1, 64));
  while (mask) {
    int from = __builtin_ctzll(mask);
    if (__popcll(mask) > 4) {
      uint64_t least = mask >> lane & 1 ? key : ~0ull;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const uint64_t w = __shfl_xor(least, o, 64);
        least = w < least ? w : least;
      }
      from = __builtin_ctzll(__ballot(key == least) & mask);
    }
    const uint64_t in = __shfl(key, from, 64);
    const int pos = __popcll(__ballot(best < in));
    const uint64_t up = __shfl_up(best, 1, 64);
    best = lane < pos ? best : (lane == pos ? in : up);
    mask &= ~(1ull << from);
    mask &= __ballot(key < __shfl(best, k - 1, 64));   // those that still can be among them
  }
}

__device__ __forceinline__ void put_answer(uint64_t best, int64_t q, int lane, int k, int32_t *out_idx,
                                           float *out_dist) {
  if (lane >= k) return;
  out_idx[q * k + lane] = best == ~0ull ? -1 : (int32_t)(uint32_t)best;
  if (out_dist) out_dist[q * k + lane] = best == ~0ull ? FLT_MAX : __uint_as_float((uint32_t)(best >> 32));
}

// ---- the band: queries whose list certifies nothing -----------------------------
//
// All candidates whose value may be an answer's are collected by the filter's
// products and ranked by their exact distances.  The values' error grows with the
// rows' norms, so those queries are put into tiles by their nearest of kPivots rows
// and a tile has a centre m of its own, one of its queries: with u = q - m,
//     |q - c|^2 = |u|^2 + 2 u.m' - 2 (u.c' - |c - m|^2 / 2)
// (m' and c' as the candidates' images are centred), and the value u.c' - |c - m|^2
// / 2 has an error of |u| |c'| and |c - m|^2, for those that matter a small share of
// what it is in the candidates' own centring.  The start values are FP32 distances
// to the tile's centre.  With points in tight clusters (100,000 x 100, distances 1/60
// of the offsets) one product leaves a few hits to a query, where in the common
// centring three left a thousand.
constexpr int kPivots = 1024;
constexpr int kBandSome = 512;   // hits ranked of a query with too many

__global__ void knn_pivot_rows_kernel(const float *__restrict__ X, int64_t M, int N, int P, float *__restrict__ pivots) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < (int64_t)P * N) pivots[e] = X[(e / N) * M / P * N + e % N];
}

// the pivots' queries counted, a block to kPivotChunk of them, in LDS first
constexpr int kPivotChunk = 4096;
__global__ void __launch_bounds__(kPivots) knn_pivot_count_kernel(const int32_t *__restrict__ rows, int64_t n,
                                                                  const int32_t *__restrict__ pivot_of,
                                                                  int32_t *__restrict__ count) {
  __shared__ int32_t here[kPivots];
  const int t = threadIdx.x;
  here[t] = 0;
  __syncthreads();
  const int64_t i0 = (int64_t)blockIdx.x * kPivotChunk, i1 = i0 + kPivotChunk < n ? i0 + kPivotChunk : n;
  for (int64_t i = i0 + t; i < i1; i += kPivots) atomicAdd(&here[pivot_of[rows[i]]], 1);
  __syncthreads();
  if (here[t]) atomicAdd(&count[t], here[t]);
}

// count[p] -> the first slot of pivot p's queries, in whole tiles; *total: all slots
__global__ void __launch_bounds__(kPivots) knn_pivot_slots_kernel(int32_t *__restrict__ count, int P,
                                                                  int32_t *__restrict__ total) {
  __shared__ int32_t at[kPivots];
  const int t = threadIdx.x;
  const int32_t mine = t < P ? (count[t] + FT - 1) / FT * FT : 0;
  at[t] = mine;
  for (int o = 1; o < kPivots; o *= 2) {
    __syncthreads();
    const int32_t w = t >= o ? at[t - o] : 0;
    __syncthreads();
    at[t] += w;
  }
  if (t < P) count[t] = at[t] - mine;
  if (t == kPivots - 1) *total = at[t];
}

// each query to a slot of its pivot's (next: the first that is free)
__global__ void __launch_bounds__(kPivots) knn_pivot_place_kernel(const int32_t *__restrict__ rows,
                                                                  const float *__restrict__ dist, int64_t n,
                                                                  const int32_t *__restrict__ pivot_of,
                                                                  int32_t *__restrict__ next,
                                                                  int32_t *__restrict__ slot_row,
                                                                  float *__restrict__ slot_dist) {
  __shared__ int32_t here[kPivots];
  const int t = threadIdx.x;
  here[t] = 0;
  __syncthreads();
  const int64_t i0 = (int64_t)blockIdx.x * kPivotChunk, i1 = i0 + kPivotChunk < n ? i0 + kPivotChunk : n;
  for (int64_t i = i0 + t; i < i1; i += kPivots) atomicAdd(&here[pivot_of[rows[i]]], 1);
  __syncthreads();
  if (here[t]) here[t] = atomicAdd(&next[t], here[t]);
  __syncthreads();
  for (int64_t i = i0 + t; i < i1; i += kPivots) {
    const int32_t at = atomicAdd(&here[pivot_of[rows[i]]], 1);
    slot_row[at] = rows[i];
    slot_dist[at] = dist[i];
  }
}

// a tile's centre: its first query (whole tiles to a pivot, so there is one)
__global__ void __launch_bounds__(256) knn_centre_kernel(const float *__restrict__ Q, int N,
                                                         const int32_t *__restrict__ slot_row, int64_t pitch,
                                                         float *__restrict__ centres) {
  const float *q = Q + (int64_t)slot_row[(int64_t)blockIdx.x * FT] * N;
  for (int n = threadIdx.x; n < N; n += 256) centres[blockIdx.x * pitch + n] = q[n];
}

// limits[slot]: the least value of a candidate as near as dist (the k-th distance
// found); -INFINITY: none, every candidate may be; INFINITY: an empty slot.  A
// wavefront to a slot, in FP64.
__global__ void __launch_bounds__(256) knn_limit_kernel(const float *__restrict__ Q, int N, int64_t slots,
                                                        const int32_t *__restrict__ slot_row,
                                                        const float *__restrict__ slot_dist,
                                                        const float *__restrict__ centres, int64_t pitch,
                                                        const float *__restrict__ mean, const float *__restrict__ unorm,
                                                        const float *__restrict__ ures, const KnnStats *__restrict__ xs,
                                                        float scale, double sub, int nseg, float *__restrict__ limits) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= slots) return;
  if (slot_row[t] < 0) {
    if (lane == 0) limits[t] = INFINITY;
    return;
  }
  const float *q = Q + (int64_t)slot_row[t] * N, *m = centres + t / FT * pitch;
  double uu = 0.0, um = 0.0, mm = 0.0;
  for (int n = lane; n < N; n += 64) {
    const double u = ((double)q[n] - (double)m[n]) * scale, v = ((double)m[n] - (double)mean[n]) * scale;
    uu += u * u;
    um += u * v;
    mm += v * v;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    uu += __shfl_xor(uu, o, 64);
    um += __shfl_xor(um, o, 64);
    mm += __shfl_xor(mm, o, 64);
  }
  if (lane > 0) return;
  const double nerr = sum_error(N), sc2 = (double)scale * scale;
  const double dist = sqrt(scaled_above(slot_dist[t], N, sc2)) * kUp;
  const double u = sqrt(uu) * kUp, ur = sqrt((double)ures[t] * (1 + nerr)) * kUp;
  const double w = u + dist, x = (sqrt(mm) + w) * kUp;   // the candidates' distance to m, and norm
  const double err = product_error(N, sub, u, ur, x, residual_at(xs, x, nerr), u * x + 0.5 * w * w, nseg) +
                     0.5 * ((N + 16) * kU23 * w * w + N * 1.5e-45 * sc2);   // the start value's own
  const double least = 0.5 * (uu + 2.0 * um - dist * dist) - err - 1e-11 * (uu + sqrt(uu * mm));
  const float f = (float)(least - 1.2e-7 * fabs(least));
  limits[t] = f > kNoValue && f < INFINITY ? f : -INFINITY;
}

// FP32 squared distances of x to the NQ rows q, which the wavefront shares: the
// additions of exact_distance, in its order
constexpr int kBruteQ = 8;

typedef const __attribute__((address_space(4))) float *ScalarRow;   // read-only, at an address the wavefront shares

template <int NQ, typename Row>
__device__ __forceinline__ void shared_distances(const float *__restrict__ x, Row q, int N, bool vec4, float (&d)[NQ]) {
#pragma unroll
  for (int f = 0; f < NQ; ++f) d[f] = 0.f;
  // CH features at a time, their loads on their way together
  auto chunk = [&](int kk, auto ch, auto vec) __attribute__((always_inline)) {
    constexpr int CH = decltype(ch)::value;
    float v[CH];
    if constexpr (decltype(vec)::value) {
#pragma unroll
      for (int j = 0; j < CH; j += 4) {
        const float4 w = *reinterpret_cast<const float4 *>(x + kk + j);
        v[j] = w.x;
        v[j + 1] = w.y;
        v[j + 2] = w.z;
        v[j + 3] = w.w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < CH; ++j) v[j] = x[kk + j];
    }
#pragma unroll
    for (int f = 0; f < NQ; ++f)
#pragma unroll
      for (int j = 0; j < CH; ++j) {
        const float w = q(f)[kk + j] - v[j];
        d[f] = fmaf(w, w, d[f]);
      }
  };
  int kk = 0;
  if (vec4) {
    for (; kk + 32 <= N; kk += 32) chunk(kk, std::integral_constant<int, 32>{}, std::true_type{});
    for (; kk < N; kk += 4) chunk(kk, std::integral_constant<int, 4>{}, std::true_type{});
  } else {
    for (; kk + 8 <= N; kk += 8) chunk(kk, std::integral_constant<int, 8>{}, std::false_type{});
    for (; kk < N; ++kk) chunk(kk, std::integral_constant<int, 1>{}, std::false_type{});
  }
}

// start values of every candidate for each of `tiles` query tiles: minus half its
// squared distance to the tile's centre; NQ tiles to a block, so that a
// candidate's row is read once for them (1,000,000 x 784, 32 tiles: 3.9 ms with
// eight, bound by the rows' way from memory, 2.3 with 32); eight where that leaves
// CUs idle (20,000 x 500: 2.7 ms the whole call, 3.1 with 32)
template <int NQ>
__global__ void __launch_bounds__(256) knn_start_kernel(const float *__restrict__ X, int64_t M, int N,
                                                        const int32_t *__restrict__ order,
                                                        const float *__restrict__ centres, int64_t pitch, int tiles,
                                                        float scale, int64_t start_pitch, float *__restrict__ start) {
  const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int b0 = blockIdx.y * NQ, nb = tiles - b0 < NQ ? tiles - b0 : NQ;
  const ScalarRow m = (ScalarRow)(centres + b0 * pitch);
  float d[NQ];
  shared_distances<NQ>(X + (int64_t)order[c < M ? c : M - 1] * N, [&](int f) { return m + (f < nb ? f : 0) * pitch; }, N,
                       rows_are_vec4(X, X, N), d);
#pragma unroll
  for (int f = 0; f < NQ; ++f)
    if (f < nb) start[(b0 + f) * start_pitch + c] = c < M ? -0.5f * (d[f] * scale) * scale : kPadStart;
}

// The slots' k nearest of their hits.  One without a limit, or with k equal points
// among more hits than were kept, goes to `all` (every candidate), one with more
// hits otherwise to `next` ([0] its count, then rows, next_dist; NULL: to all), with
// the k-th distance of some of them: of a thousand points of a cluster the k nearest
// are much nearer than of the list's eight.
// Bound by the latency of the hits' rows, which come from L2 and the memory-side
// cache, so the four waves of a block share a query (a wave to a query: 100,000 x
// 100 points with 5,000 hits each 28 ms).
__global__ void __launch_bounds__(256) knn_band_rank_kernel(const float *__restrict__ X, int N,
                                                            const float *__restrict__ Q,
                                                            const int32_t *__restrict__ slot_row,
                                                            const float *__restrict__ slot_dist,
                                                            const float *__restrict__ limits,
                                                            const int32_t *__restrict__ count,
                                                            const int32_t *__restrict__ ids, int cap,
                                                            const int32_t *__restrict__ order, int k,
                                                            int32_t *__restrict__ out_idx,
                                                            float *__restrict__ out_dist, int32_t *__restrict__ all,
                                                            int32_t *__restrict__ next, float *__restrict__ next_dist) {
  __shared__ uint64_t lists[4][32];
  static_assert(sizeof lists / sizeof lists[0][0] == 4 * 32, "k is at most 28");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t t = blockIdx.x, q = slot_row[t];
  if (q < 0) return;
  const int32_t hits = count[t];
  const bool over = hits > cap;
  if (!(limits[t] > -INFINITY) || (over && (!next || slot_dist[t] == 0.f))) {
    if (threadIdx.x == 0) all[1 + atomicAdd(&all[0], 1)] = (int32_t)q;
    return;
  }
  const int32_t n = over ? kBandSome : hits;   // (past cap - 64 places may not be written)
  const bool vec4 = rows_are_vec4(X, Q, N);
  uint64_t best = ~0ull;
  for (int32_t base = 64 * wave; base < n; base += 256) {
    uint64_t key = ~0ull;
    if (base + lane < n) {
      const int32_t c = order[ids[t * cap + base + lane]];
      key = (uint64_t)__float_as_uint(exact_distance(Q + q * N, X + (int64_t)c * N, N, vec4)) << 32 | (uint32_t)c;
    }
    offer_sorted(best, key, lane, k);
  }
  if (lane < 32) lists[wave][lane] = best;
  __syncthreads();
  if (wave > 0) return;
  for (int w = 1; w < 4; ++w) offer_sorted(best, lane < k ? lists[w][lane] : ~0ull, lane, k);
  if (!over) {
    put_answer(best, q, lane, k, out_idx, out_dist);
  } else if (lane == k - 1) {
    const int32_t at = atomicAdd(&next[0], 1);
    next[1 + at] = (int32_t)q;
    next_dist[at] = fminf(slot_dist[t], __uint_as_float((uint32_t)(best >> 32)));
  }
}

// Every candidate.  A block takes kBruteQ queries over one range of the
// candidates: thread t computes the FP32 distances of candidate c0 + t (a tile of
// 256 at a time) to all of them, 32 features of its row in registers and the
// queries' through the scalar cache; the four waves then offer the tile's keys to
// two queries each.  Bound by the vector ALU (2 instructions per query, candidate
// and feature).  A range ends when k candidates of distance 0 are found for each
// query: those that follow have higher ids.
__global__ void __launch_bounds__(256) knn_brute_kernel(const float *__restrict__ X, int64_t M, int N,
                                                        const float *__restrict__ Q, int64_t nq,
                                                        const int32_t *__restrict__ rows, int self_mode,
                                                        const int32_t *__restrict__ self, int k, int splits,
                                                        uint64_t *__restrict__ part, int32_t *__restrict__ out_idx,
                                                        float *__restrict__ out_dist) {
  __shared__ uint64_t keys[kBruteQ][256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t f0 = (int64_t)blockIdx.x * kBruteQ;
  const int nf = nq - f0 < kBruteQ ? (int)(nq - f0) : kBruteQ;
  const int64_t per = ((M + splits - 1) / splits + 255) / 256 * 256;
  const int64_t b = blockIdx.y * per, e = b + per < M ? b + per : M;
  const bool vec4 = rows_are_vec4(X, Q, N);
  ScalarRow qrow[kBruteQ];
  int64_t own[kBruteQ];
#pragma unroll
  for (int f = 0; f < kBruteQ; ++f) {
    const int64_t at = f0 + (f < nf ? f : 0), q = rows ? (int64_t)rows[at] : at;
    qrow[f] = (ScalarRow)(Q + q * N);
    own[f] = self_mode == 1 ? q : (self_mode == 2 ? (int64_t)self[q] : -1);
  }
  uint64_t best[2] = {~0ull, ~0ull};
  for (int64_t c0 = b; c0 < e; c0 += 256) {
    const int64_t c = c0 + tid;
    const float *x = X + (c < e ? c : e - 1) * N;
    float d[kBruteQ];
    shared_distances<kBruteQ>(x, [&](int f) { return qrow[f]; }, N, vec4, d);
#pragma unroll
    for (int f = 0; f < kBruteQ; ++f)
      keys[f][tid] = c < e && f < nf && c != own[f] ? (uint64_t)__float_as_uint(d[f]) << 32 | (uint32_t)c : ~0ull;
    __syncthreads();
    bool done = true;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      for (int g = 0; g < 4; ++g) offer_sorted(best[h], keys[2 * wave + h][64 * g + lane], lane, k);
      done = done && (2 * wave + h >= nf || __shfl(best[h], k - 1, 64) >> 32 == 0);
    }
    if (__syncthreads_and(done)) break;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int64_t f = f0 + 2 * wave + h;
    if (f >= nq) continue;
    if (splits == 1) put_answer(best[h], rows ? (int64_t)rows[f] : f, lane, k, out_idx, out_dist);
    else if (lane < k) part[(f * splits + blockIdx.y) * k + lane] = best[h];
  }
}

// one wavefront per query: the k best of its ranges' lists
__global__ void __launch_bounds__(256) knn_brute_merge_kernel(const uint64_t *__restrict__ part, int64_t nq,
                                                              const int32_t *__restrict__ rows, int k, int splits,
                                                              int32_t *__restrict__ out_idx,
                                                              float *__restrict__ out_dist) {
  const int lane = threadIdx.x & 63;
  const int64_t f = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (f >= nq) return;
  uint64_t best = ~0ull;
  const uint64_t *P = part + f * splits * k;
  for (int base = 0; base < splits * k; base += 64)
    offer_sorted(best, base + lane < splits * k ? P[base + lane] : ~0ull, lane, k);
  put_answer(best, rows ? (int64_t)rows[f] : f, lane, k, out_idx, out_dist);
}

template <int KP, bool SEG3>
hipError_t launch_filter_kp(const FilterArgs &f, const FinishArgs &g, hipStream_t s) {
  knn_filter_kernel<KP, SEG3, false><<<(unsigned)(f.nqb * f.splits), kFilterThreads, 0, s>>>(f);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  knn_finish_kernel<KP><<<grid_for(g.n_launch * KP, 256), 256, 0, s>>>(g);
  return hipGetLastError();
}

// candidate ranges per query tile: the number that gives the shortest
// schedule on 256 CUs (one block each).  A tile costs about 0.9 us per stage
// and 0.7 us for its values; a range costs about 40 us for its hits and their
// lists, whatever its length, and each list it leaves 0.1 ns per entry to merge.
int choose_splits(int64_t nqb, int64_t tiles, int stages, int kp) {
  int best = 1;
  double best_t = 1e300;
  for (int s = 1; s <= 64 && s <= tiles; ++s) {
    const int64_t rounds = (nqb * s + kCus - 1) / kCus, per = (tiles + s - 1) / s;
    const double t = (double)rounds * ((double)per * (0.9 * stages + 0.7) + 40.0) + 1e-4 * (double)nqb * FT * s * kp;
    if (t < best_t * 0.995) {
      best_t = t;
      best = s;
    }
  }
  return best;
}

// tiles of a range that set its starting thresholds: about a thirtieth of it,
// but all of a short one (its hits are then little more than the list)
int lead_tiles(int64_t tiles) {
  return (int)(tiles <= 4 ? tiles : (tiles < 64 ? 3 + tiles / 16 : (tiles < 1024 ? tiles / 32 + 5 : 37)));
}

hipError_t run_filter(const FilterArgs &f, const FinishArgs &g, int kp, hipStream_t s) {
  const bool three = g.nseg == 3;
  switch (kp) {
    case 8: return three ? launch_filter_kp<8, true>(f, g, s) : launch_filter_kp<8, false>(f, g, s);
    case 16: return three ? launch_filter_kp<16, true>(f, g, s) : launch_filter_kp<16, false>(f, g, s);
    default: return three ? launch_filter_kp<32, true>(f, g, s) : launch_filter_kp<32, false>(f, g, s);
  }
}

// the shortest list with room for candidates that a misranks
int list_length(int k) { return k + 4 <= 8 ? 8 : (k + 4 <= 16 ? 16 : 32); }

// query tiles of one launch (a multiple of the CUs; bounds the lists' memory)
constexpr int64_t kBatchTiles = 16 * kCus;

int64_t knn_image_halves(int64_t M, int N) { return (M + FT - 1) / FT * FT * (int64_t)((N + FK - 1) / FK * FK); }

// (an image without room for the rows is refused)
hipError_t launch_knn_split(const float *X, int64_t M, int N, const int32_t *map, const float *mean,
                            int64_t mean_stride, float scale, const KnnImage &hi, const KnnImage &lo, float *norms, float *res,
                            float *start, KnnStats *stats, hipStream_t s) {
  const int64_t need = knn_image_halves(M, N);
  if ((hi.p && need > hi.halves) || (lo.p && need > lo.halves)) return hipErrorInvalidValue;
  const bool vec = N % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0;   // (the centres are aligned)
  const int64_t groups = (M + FT - 1) / FT * (FT / 16);
  knn_split_kernel<<<(unsigned)(groups < 4096 ? groups : 4096), 256, 0, s>>>(
      X, M, N, (N + FK - 1) / FK, map, mean, mean_stride, scale, hi.p, lo.p, norms, res, start, stats, vec);
  return hipGetLastError();
}

// Power of two for a sample of that spread: it below 2^8, so that values 256 times
// as large are in range and values 2^-22 of it on the normal FP16 grid; |s| <= 126, so that the scale and its
// inverse are normal floats.  spread 0: any finite magnitude in range.
float sample_scale(float spread, float absmax) {
  if (!(absmax > 0.f)) return 1.f;
  const bool some = spread > 0.f && std::isfinite(spread);
  int e;
  (void)frexpf(some ? spread : absmax, &e);   // m 2^e, 0.5 <= m < 1
  int sh = (some ? 8 : 14) - e;
  sh = sh > 126 ? 126 : (sh < -126 ? -126 : sh);
  return ldexpf(1.f, sh);
}

// List length: the pilot runs kPilotTiles query tiles spread over the call and
// counts the answers that lists of 8, 16 and (when k asks for those anyway) 32
// would not certify.  A tile costs its products (as in choose_splits), those again
// and a little for the share that fails (the band), and, more for a longer list, its
// hits: kListCost, in the same us (at 400,000 x 100 lists of 8, 16 and 32 sweep in
// 62, 74 and about 90 ms, against 45 ms without any hit); the cheapest is taken.
// Calls of fewer query tiles than CUs go without a pilot, which takes as long as it
// takes a block to fill its lists (1.4 ms with lists of 32) and leaves most CUs
// idle: 50,000 x 128, k 2 / 5 / 10 / 20: 2.8 / 3.4 / 5.0 / 7.3 ms with one, 2.4 / 2.7
// / 3.9 / 5.9 without.  Wide rows keep it from 4 kPilotTiles tiles on, as their
// failed answers cost more than the pilot (20,000 x 500, k 10: 2.9 ms with it, 3.6
// without).  With fewer than kFewTiles candidate tiles (a coarse quantizer's
// centroids) the lists cost more than the products, so short lists and three
// segments are best (200,000 queries against 512 centroids of width 100).
constexpr double kListCost[3] = {1.6, 2.8, 4.3};
constexpr int kWidePilot = 256;
constexpr int64_t kPilotTiles = 8;
constexpr int64_t kFewTiles = 16;

// Ranges of the candidates, for blocks of kBruteQ queries: to fill the chip
int64_t brute_splits(int64_t nq, int64_t M) {
  const int64_t groups = (nq + kBruteQ - 1) / kBruteQ, tiles = (M + 255) / 256;
  int64_t splits = 4 * kCus / groups;
  splits = splits < 1 ? 1 : (splits > 256 ? 256 : splits);
  return splits < tiles ? splits : tiles;
}

// Whether a call's exact distances take no longer than the filter and what goes
// with it.  In us, fitted to calls of 100 to 200,000 candidates, 1 to 200,000
// queries, 2 to 784 features and k 1, 5 and 28, so that it errs towards the filter:
// the filter takes 310 (600 with lists of 32) against few candidates, else 520
// (1,500), for a query's list 2 to 11 ns, for the operands 12 ps a feature of a
// query and 6 of a candidate, and for a pair of tiles as in choose_splits; the
// distances take 110, 64 fs a pair and feature (81 % of the vector ALU) and as much
// as 17 features for a pair's way through the lists.  300 x 3, k 2: 273 -> 97 us
// (195 with the search before the filter); 128 x 64 and 50,000 queries: 356 -> 194
// (252); 1,000 x 20, k 5: 307 -> 109 (764).
bool direct_pays(int64_t M, int N, int64_t nq, int k, bool few, bool same) {
  const double pairs = (double)((nq + kBruteQ - 1) / kBruteQ * kBruteQ) * (double)((M + 255) / 256 * 256);
  const double blocks = (double)((nq + kBruteQ - 1) / kBruteQ) * (double)brute_splits(nq, M);
  const double idle = blocks < 4 * kCus ? 4 * kCus / blocks : 1.0;
  const double stages = (double)((N + FK - 1) / FK) * (few ? 3 : 1);
  const double filter = (few ? (k > 12 ? 600.0 : 310.0) : (k > 12 ? 1500.0 : 520.0)) +
                        (double)nq * (k > 12 ? 1.1e-2 : (k > 4 ? 3e-3 : 1.9e-3)) + 1.2e-5 * (double)nq * N +
                        (same ? 0.0 : 6e-6 * (double)M * N) +
                        pairs * (0.9 * stages + 0.7) / (FT * FT * (double)kCus);
  const double direct = 110.0 + 6.4e-8 * pairs * (N + 17) * idle + 2.7e-6 * (double)nq * N;
  return direct <= filter;
}

// The band's hits: so many are kept of a query with one segment and with three,
// and so many in all, with the start values of a batch (they fit buffers that the
// library keeps)
constexpr int64_t kBandHits[2] = {4096, 16384};
static_assert(kBandHits[0] - 64 >= kBandSome, "hits that are ranked are there");
constexpr int64_t kBandIds = int64_t{32} << 20;

}  // namespace

// x with a x = 1 mod m (a prime to m)
static int64_t inverse_mod(int64_t a, int64_t m) {
  int64_t r0 = m, r1 = a % m, x0 = 0, x1 = 1;
  while (r1) {
    const int64_t q = r0 / r1, r = r0 - q * r1, x = x0 - q * x1;
    r0 = r1;
    r1 = r;
    x0 = x1;
    x1 = x;
  }
  return (x0 % m + m) % m;
}

int KnnSearch::open(int64_t M_, int N_, const float *Q_, int64_t nq_, const float *sample, int64_t sample_rows,
                    bool same_, int k_, hipStream_t s_) {
  M = M_;
  N = N_;
  Q = Q_;
  nq = nq_;
  same = same_;
  k = k_;
  s = s_;
  S.stream = s_;
  few = (M + FT - 1) / FT < kFewTiles;
  direct = direct_pays(M, N, nq, k, few, same);
  const int64_t tiles = (M + FT - 1) / FT, nx = knn_image_halves(M, N), nqi = knn_image_halves(nq, N);
  Carve V;
  auto image = [&](KnnImage *im, int64_t halves) {
    V.add(&im->p, halves);
    im->halves = halves;
  };
  uint32_t *spread = nullptr;   // of the sample, then the largest |coordinate|
  V.add(&spread, 2);
  if (!direct) {
    image(&ch, nx);
    V.add(&start, tiles * FT);
    V.add(&xstats, 1);
    V.add(&fails, nq + 1);
    V.add(&fail_dist, nq);
    V.add(&pilot, 3);
    V.add(&mean, N);
    V.add(&qnorm, nq);
    V.add(&qres, nq);
    V.add(&order, M);
    if (few) image(&cl, nx);
    if (!same) {
      image(&qh, nqi);
      if (few) image(&ql, nqi);
    }
  }
  const int rc = V.get(S, "operands of the search");
  if (rc) return rc;
  if (same) {
    qh = ch;
    ql = cl;
  }
  uint32_t bits[2];
  float seen[2];
  HIPCHK(launch_fill_i32((int32_t *)spread, 2, 0, s));
  HIPCHK(launch_absmax(sample, sample_rows * N, spread + 1, s));
  if (Q != sample || nq != sample_rows) HIPCHK(launch_absmax(Q, nq * N, spread + 1, s));
  if (!direct) {
    int64_t stride = (int64_t)((double)M * 0.6180339887498949);
    while (stride < 1 || std::gcd(stride, M) != 1) ++stride;
    place_of = inverse_mod(stride, M);
    knn_order_kernel<<<grid_for(M), kBlock, 0, s>>>(M, stride, order);
    knn_sample_kernel<<<(unsigned)N, 256, 0, s>>>(sample, sample_rows, N, mean, spread);
  }
  HIPCHK(hipGetLastError());
  HIPCHK(hipMemcpyAsync(bits, spread, sizeof bits, hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  std::memcpy(seen, bits, sizeof bits);
  if (!std::isfinite(seen[1])) return fail(IVHD_EINVAL, "the points hold a non-finite coordinate");
  scale = sample_scale(seen[0], seen[1]);
  return IVHD_OK;
}

int KnnSearch::run(const float *X, int self_mode, const int32_t *self, int32_t *idx, float *dist) {
  if (direct) return rank_all(X, nullptr, nq, self_mode, self, idx, dist);
  const int nk = (N + FK - 1) / FK;
  const int64_t tiles = (M + FT - 1) / FT, nqb = (nq + FT - 1) / FT;
  int kp = list_length(k), rc;
  HIPCHK(launch_fill_i32((int32_t *)xstats, sizeof(KnnStats) / 4, 0, s));
  HIPCHK(launch_knn_split(X, M, N, order, mean, 0, scale, ch, cl, same ? qnorm : nullptr, same ? qres : nullptr, start,
                          xstats, s));
  knn_classes_kernel<<<1, kNormClasses, 0, s>>>(xstats, N);
  HIPCHK(hipGetLastError());
  if (!same && !queries_ready) {
    HIPCHK(launch_knn_split(Q, nq, N, nullptr, mean, 0, scale, qh, ql, qnorm, qres, nullptr, nullptr, s));
    queries_ready = true;   // their images do not depend on the candidates
  }

  FilterArgs f{};
  f.Qh = qh.p;
  f.Ql = ql.p;
  f.Ch = ch.p;
  f.Cl = cl.p;
  f.start = start;
  f.nk = nk;
  f.nq = nq;
  f.tiles = tiles;
  f.M = M;
  f.place_of = place_of;
  f.map = same ? order : nullptr;
  f.self_mode = self_mode;
  f.self = self;
  FinishArgs g{};
  g.X = X;
  g.Q = Q;
  g.N = N;
  g.nk = nk;
  g.k = k;
  g.nq = nq;
  g.M = M;
  g.map = f.map;
  g.order = order;
  g.self_mode = self_mode;
  g.self = self;
  g.out_idx = idx;
  g.out_dist = dist;
  g.nseg = few ? 3 : 1;   // few candidates: both halves are made at once
  g.qnorm = qnorm;
  g.qres = qres;
  g.xs = xstats;
  g.sub = 3e-8 * std::sqrt((double)N);
  g.scale = scale;
  g.fails = fails;
  g.fail_dist = fail_dist;

  // the query tiles qb0, qb0 + step, .., of images `images`
  auto shape = [&](int64_t qb0, int64_t step, int64_t n, int nseg, int list, const KnnImage &images) -> int {
    f.qb0 = g.qb0 = qb0;
    f.qb_step = g.qb_step = step;
    f.nqb = n;
    f.splits = g.splits = choose_splits(n, tiles, nk * nseg, list);
    f.tiles_per_split = (tiles + f.splits - 1) / f.splits;
    f.lead = lead_tiles(f.tiles_per_split);
    g.n_launch = n * FT;
    if ((qb0 + (n - 1) * step + 1) * nk * kTileHalves > images.halves || tiles * nk * kTileHalves > ch.halves)
      return fail(IVHD_ESTATE, "kNN: query tiles outside their operands");
    return IVHD_OK;
  };
  auto sweep = [&](int64_t qb0, int64_t step, int64_t n) -> int {
    int r = shape(qb0, step, n, g.nseg, kp, qh);
    if (r) return r;
    const int64_t need = n * FT * f.splits * kp;
    if (need > part_cap) {   // (a larger launch is queued behind the smaller: both lists stay)
      if ((r = S.get(&part, need, "candidate lists"))) return r;
      part_cap = need;
    }
    f.part = part;
    g.part = part;
    HIPCHK(run_filter(f, g, kp, s));
    return IVHD_OK;
  };
  if (!few && nqb >= (N > kWidePilot ? 4 * kPilotTiles : kCus)) {
    int32_t bad[3];
    HIPCHK(launch_fill_i32(pilot, 3, 0, s));
    g.pilot = pilot;
    const int want = kp;
    kp = kp < 16 ? 16 : kp;
    if ((rc = sweep(0, nqb / kPilotTiles, kPilotTiles))) return rc;
    g.pilot = nullptr;
    HIPCHK(hipMemcpyAsync(bad, pilot, sizeof bad, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    double least = 1e300;
    for (int l = want == 8 ? 0 : (want == 16 ? 1 : 2); l < 3; ++l) {
      const bool seen = (8 << l) <= (want == 32 ? 32 : 16);   // else, of 32: a third, or as many if half fail with 16
      const double share = bad[seen ? l : 1] / (double)(kPilotTiles * FT);
      const double fails = seen || share > 0.5 ? share : share / 3;
      const double cost = kListCost[l] + (0.9 * nk + 0.7) * (1 + 1.2 * fails);
      if (cost < least) {
        least = cost;
        kp = 8 << l;
      }
    }
  } else if (!few && kp == 8) {
    kp = 16;
  }
  HIPCHK(launch_fill_i32(fails, 1, 0, s));
  // all query tiles: whole rounds of the CUs take the candidates in one range,
  // which costs the fewest hits; the rest is split to fill the CUs once more
  // (few candidates: one launch, a second would last as long as a round)
  const int64_t whole = few ? nqb : nqb / kCus * kCus;
  for (int64_t b = 0; b < whole; b += kBatchTiles)
    if ((rc = sweep(b, 1, whole - b < kBatchTiles ? whole - b : kBatchTiles))) return rc;
  if (nqb > whole && (rc = sweep(whole, 1, nqb - whole))) return rc;
  auto read_count = [&](const int32_t *list, int32_t *n) -> int {
    HIPCHK(hipMemcpyAsync(n, list, sizeof *n, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    return IVHD_OK;
  };
  int32_t failed = 0;
  if ((rc = read_count(fails, &failed)) || failed == 0) return rc;

  // The answers that are not certified: every candidate where that is less than the
  // band's launches and sweeps (in us, as in direct_pays; 100,000 queries left of a
  // search in 512 x 60 candidates: 0.3 ms against 1.3), else the band, with one
  // segment, then with three for those that leave too many hits; then every candidate
  if (6.4e-8 * failed * (double)M * (N + 17) <
      500.0 + 5e-3 * failed + (double)failed / FT * (double)tiles * (0.9 * nk + 0.7) / (double)kCus)
    return rank_all(X, fails + 1, failed, self_mode, self, idx, dist);
  Scratch R(s);   // of this run
  KnnImage low_c = cl;
  int32_t *all, *next[2], *pivot_of;
  float *next_dist[2], *pivots;
  if ((rc = R.get(&all, (int64_t)failed + 1, "queries for all candidates")) || (rc = R.get(&pivot_of, nq, "queries' pivots")) ||
      (rc = R.get(&pivots, (int64_t)kPivots * N, "pivots")) || (rc = R.get(&next[1], (int64_t)failed + 1, "queries left")) ||
      (rc = R.get(&next_dist[1], failed, "their distances")))
    return rc;
  next[0] = fails;
  next_dist[0] = fail_dist;
  HIPCHK(launch_fill_i32(all, 1, 0, s));
  HIPCHK(launch_fill_i32(next[1], 1, 0, s));
  for (int pass = 0; pass < 2 && failed > 0; ++pass) {
    const int segs = pass ? 3 : 1;
    const int32_t *rows = next[pass] + 1;
    // pivots: so many that their tiles' empty places are a quarter at most; one
    // where those would tell little apart, but for the queries that one segment
    // left with too many hits
    int64_t P = failed / (2 * FT);
    P = P < (pass ? 64 : 16) ? (pass ? 64 : 1) : (P > kPivots ? kPivots : P);
    if (P > M) P = M;
    Scratch B(s);   // of this pass
    // the queries by pivots, in whole tiles
    int32_t *slots_of, *slot_row, total = 0;
    float *slot_dist;
    const int64_t room = failed + P * (FT - 1);
    if ((rc = B.get(&slots_of, kPivots + 1, "slots of the pivots")) || (rc = B.get(&slot_row, room, "slots' queries")) ||
        (rc = B.get(&slot_dist, room, "slots' distances")))
      return rc;
    if (P > 1) {
      knn_pivot_rows_kernel<<<grid_for(P * N), kBlock, 0, s>>>(X, M, N, (int)P, pivots);
      knn_brute_kernel<<<(unsigned)((failed + kBruteQ - 1) / kBruteQ), 256, 0, s>>>(
          pivots, P, N, Q, failed, rows, 0, nullptr, 1, 1, nullptr, pivot_of, nullptr);
    } else {
      HIPCHK(launch_fill_i32(pivot_of, nq, 0, s));
    }
    HIPCHK(launch_fill_i32(slots_of, kPivots + 1, 0, s));
    HIPCHK(launch_fill_i32(slot_row, room, -1, s));
    knn_pivot_count_kernel<<<grid_for(failed, kPivotChunk), kPivots, 0, s>>>(rows, failed, pivot_of, slots_of);
    knn_pivot_slots_kernel<<<1, kPivots, 0, s>>>(slots_of, (int)P, slots_of + kPivots);
    knn_pivot_place_kernel<<<grid_for(failed, kPivotChunk), kPivots, 0, s>>>(rows, next_dist[pass], failed, pivot_of,
                                                                             slots_of, slot_row, slot_dist);
    HIPCHK(hipGetLastError());
    if ((rc = read_count(slots_of + kPivots, &total))) return rc;
    const int64_t qtiles = total / FT, pitch = (N + 3) / 4 * 4;
    // their operands
    auto image = [&](KnnImage *im, int64_t n, Scratch &S, const char *what) -> int {
      im->halves = knn_image_halves(n, N);
      return S.get(&im->p, im->halves, what);
    };
    KnnImage high, low;
    float *centres, *unorm, *ures, *limits;
    if ((rc = image(&high, total, B, "query operands (high)")) ||
        (segs == 3 && (rc = image(&low, total, B, "query operands (low)"))) ||
        (rc = B.get(&centres, qtiles * pitch, "tiles' centres")) || (rc = B.get(&unorm, total, "offsets")) ||
        (rc = B.get(&ures, total, "offsets' residuals")) || (rc = B.get(&limits, total, "limits")))
      return rc;
    knn_centre_kernel<<<(unsigned)qtiles, 256, 0, s>>>(Q, N, slot_row, pitch, centres);
    HIPCHK(launch_knn_split(Q, total, N, slot_row, centres, pitch, scale, high, low, unorm, ures, nullptr, nullptr, s));
    if (segs == 3 && !low_c.p) {
      if ((rc = image(&low_c, M, R, "candidate operands (low)"))) return rc;
      HIPCHK(launch_knn_split(X, M, N, order, mean, 0, scale, KnnImage{}, low_c, nullptr, nullptr, nullptr, nullptr, s));
    }
    knn_limit_kernel<<<grid_for(total, 4), 256, 0, s>>>(Q, N, total, slot_row, slot_dist, centres, pitch, mean, unorm, ures,
                                                        xstats, scale, g.sub, segs, limits);
    HIPCHK(hipGetLastError());
    // a batch of tiles at a time: their start values, hits and answers
    const int64_t cap = M < kBandHits[pass] ? M : kBandHits[pass], start_pitch = tiles * FT;
    int64_t batch = kBandIds / (cap * FT), most = kBandIds / start_pitch;
    batch = batch < most ? batch : most;
    batch = batch < kBruteQ ? kBruteQ : batch;
    batch = batch < qtiles ? batch : qtiles;
    int32_t *count, *ids;
    float *starts;
    if ((rc = B.get(&count, batch * FT, "hits of a query")) || (rc = B.get(&ids, batch * FT * cap, "hits")) ||
        (rc = B.get(&starts, batch * start_pitch, "start values")))
      return rc;
    f.Qh = high.p;
    f.Ql = low.p;
    f.Cl = low_c.p;
    f.nq = total;
    f.map = slot_row;
    f.limits = limits;
    f.count = count;
    f.ids = ids;
    f.cap = (int)cap;
    f.start = starts;
    f.start_pitch = start_pitch;
    int32_t *to = pass ? nullptr : next[1];
    for (int64_t b = 0; b < qtiles; b += batch) {
      const int64_t n = qtiles - b < batch ? qtiles - b : batch, at = b * FT;
      if ((rc = shape(b, 1, n, segs, 0, high))) return rc;
      HIPCHK(launch_fill_i32(count, n * FT, 0, s));
      if (tiles * ((n + 31) / 32) >= 2 * kCus)
        knn_start_kernel<32><<<dim3((unsigned)tiles, (unsigned)((n + 31) / 32)), 256, 0, s>>>(
            X, M, N, order, centres + b * pitch, pitch, (int)n, scale, start_pitch, starts);
      else
        knn_start_kernel<8><<<dim3((unsigned)tiles, (unsigned)((n + 7) / 8)), 256, 0, s>>>(
            X, M, N, order, centres + b * pitch, pitch, (int)n, scale, start_pitch, starts);
      const unsigned grid = (unsigned)(f.nqb * f.splits);
      if (segs == 3) knn_filter_kernel<8, true, true><<<grid, kFilterThreads, 0, s>>>(f);
      else knn_filter_kernel<8, false, true><<<grid, kFilterThreads, 0, s>>>(f);
      knn_band_rank_kernel<<<(unsigned)(n * FT), 256, 0, s>>>(X, N, Q, slot_row + at, slot_dist + at, limits + at, count,
                                                              ids, (int)cap, order, k, idx, dist, all, to,
                                                              pass ? nullptr : next_dist[1]);
      HIPCHK(hipGetLastError());
    }
    if ((rc = read_count(next[1], &failed))) return rc;
  }
  if ((rc = read_count(all, &failed)) || failed == 0) return rc;
  return rank_all(X, all + 1, failed, self_mode, self, idx, dist);
}

int KnnSearch::rank_all(const float *X, const int32_t *rows, int64_t n, int self_mode, const int32_t *self, int32_t *idx,
                        float *dist) {
  const int64_t groups = (n + kBruteQ - 1) / kBruteQ, splits = brute_splits(n, M);
  Scratch R(s);
  uint64_t *bp = nullptr;
  int rc;
  if (splits > 1 && (rc = R.get(&bp, n * splits * k, "candidate lists (all candidates)"))) return rc;
  knn_brute_kernel<<<dim3((unsigned)groups, (unsigned)splits), 256, 0, s>>>(X, M, N, Q, n, rows, self_mode, self, k,
                                                                            (int)splits, bp, idx, dist);
  if (splits > 1) knn_brute_merge_kernel<<<grid_for(n, 4), 256, 0, s>>>(bp, n, rows, k, (int)splits, idx, dist);
  HIPCHK(hipGetLastError());
  HIPCHK(hipStreamSynchronize(s));
  return IVHD_OK;
}

}  // namespace ivhd
