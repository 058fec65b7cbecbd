// Quality of a layout on a sample of points (thesis, chapter "Quality
// metrics": Sec. "Rank-based criteria", Sec. "Neighbor hit",
// Sec. "Trustworthiness and continuity").  Off the timed path.
//
// Everything is decided by the order of the points around a sample row r:
// all M points (r itself included) sorted by (delta_rl, l) with delta the
// squared Euclidean distance, accumulated in FP64 from the FP32 coordinates
// in dimension order, ties to the lower index.  The rank rho_rj is the
// position of j in that order; the neighbourhood of size k is positions
// 1..k.  FP64 makes these integer decisions the same as a plain FP64
// evaluation of the same definition (each per-dimension term (x - y)^2 of
// two FP32 values is exact in FP64; only the additions round).
//
// One block takes kRows sample rows and one contiguous chunk of the candidates
// (blockIdx.y), a candidate per lane: what belongs to a sample row is then the
// same for all lanes and comes through the scalar cache (its coordinates, as
// FP64 [dimension][kRows], and its thresholds), and a candidate's coordinate
// is converted once for kRows distances.  FP64 adds and multiplies run at the
// rate of unpacked FP32 here, so the distances are computed in FP64 at once,
// two operations a dimension, which is what bounds more than a few
// dimensions: 2.0 ms at 39 T operations/s for 2000 rows of 200,000
// candidates in 100 dimensions.  The multiply-add is written out, so that
// every distance of a pair has the same bits in every kernel.
//
// Neighbour mode appends the pairs at or below the row's threshold to a buffer
// in LDS; a buffer that might not hold the next tile's pairs is cut back to a
// few more than the best k + 1, whose largest is the new threshold, of all the
// row's chunks (a row's k + 1 nearest are at or below each of its thresholds).
// A chunk by itself costs a row about (k + 1) ln(chunk / (k + 1)) appended
// pairs, and a cut every so many (one for each kThreads candidates at worst,
// where each is nearer than all before).
// The cut is a bisection on the pair's bits, all in registers.  Rank mode
// counts, for each of the kc thresholds, the candidates before it, by the
// lanes of a comparison.
//
// Measured, 2000 rows of 200,000 candidates, against a sample row per lane
// with its list in LDS: 100 nearest in 2 dimensions 0.52 ms (197), 10 nearest
// in 100 dimensions 5.4 ms (16.9), 10 ranks there 5.2 ms (22.7).  The vector
// units are busy for two thirds of the scans in 100 dimensions, at 1.94 GHz,
// with 1.4 instructions to each one of the distances.
#include <cfloat>
#include <climits>
#include <cmath>

#include "ivhd_internal.h"
#include "knn_internal.h"
#include "knn_rank.h"

namespace ivhd {
namespace {

constexpr int kRows = 8;            // sample rows per block
constexpr int kThreads = 256;
constexpr int kEvalWaves = kThreads / 64;
constexpr int kCand = 4;            // candidates per thread: 4 kThreads to a tile, taken up kThreads at a time
constexpr int kTile = kCand * kThreads;
constexpr int kEvalDims = 8;        // dimensions staged at a time above 8
constexpr int kEvalPad = kEvalDims + 1;
constexpr int64_t kEvalRowBytes = 64 << 20;   // rows taken at a time: their coordinates and lists within this

__device__ __forceinline__ bool pair_before(double a, int32_t ia, double b, int32_t ib) {
  return a < b || (a == b && ia < ib);
}

// read-only memory at an address that the wavefront shares: loaded by the scalar unit
typedef const __attribute__((address_space(4))) double *ScalarRows;

// the sample rows' coordinates as FP64, [group][ND][kRows]: zero past the
// last dimension, the last row again past the last row; the rows' shared
// thresholds (neighbour mode) before any candidate
__global__ void eval_rows_kernel(const float *__restrict__ Z, int N, int ND, const int32_t *__restrict__ rows,
                                 int64_t Q, double *__restrict__ rq, unsigned long long *__restrict__ row_thr) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t groups = (Q + kRows - 1) / kRows;
  if (t >= groups * kRows * ND) return;
  const int64_t slot = t / ND;
  const int d = (int)(t - slot * ND);
  const int64_t q = slot < Q ? slot : Q - 1;
  if (row_thr && d == 0 && slot < Q) row_thr[slot] = (unsigned long long)__double_as_longlong(DBL_MAX);
  rq[((slot / kRows) * ND + d) * kRows + slot % kRows] = d < N ? (double)Z[(int64_t)rows[q] * N + d] : 0.0;
}

// Squared distances of the thread's candidates t0 + c kThreads + thread to the
// block's kRows rows.  Dimensions past N add exact zeros; a candidate past the
// range reads row c1 - 1.  kCand candidates to one scalar load of a dimension
// of the rows: with one, the loads' latency (they miss the scalar cache where
// the blocks of a CU have different rows) took four fifths of the time.
template <bool STAGED, int DC>
__device__ __forceinline__ void tile_distances(const float *__restrict__ Z, int N, int ND, ScalarRows rq, uint32_t t0,
                                               uint32_t c1, float *stage, double (&acc)[kCand][kRows]) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int c = 0; c < kCand; ++c)
#pragma unroll
    for (int r = 0; r < kRows; ++r) acc[c][r] = 0.0;
  auto add = [&](int c, double zd, const double (&row)[kRows]) {
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const double t = zd - row[r];
      acc[c][r] = fma(t, t, acc[c][r]);
    }
  };
  if (!STAGED) {
    float z[kCand][DC];
#pragma unroll
    for (int c = 0; c < kCand; ++c) {
      const uint32_t at = t0 + c * kThreads + tid;
      const float *zr = Z + (int64_t)(at < c1 ? at : c1 - 1) * N;
#pragma unroll
      for (int d = 0; d < DC; ++d) z[c][d] = d < N ? zr[d] : 0.f;
    }
#pragma unroll
    for (int d = 0; d < DC; ++d) {
      if (d % 2 == 0) asm volatile("" : "+s"(rq));   // read anew: held over the tiles, they overflow the scalar registers
      double row[kRows];
#pragma unroll
      for (int r = 0; r < kRows; ++r) row[r] = rq[d * kRows + r];
#pragma unroll
      for (int c = 0; c < kCand; ++c) add(c, (double)z[c][d], row);
    }
    return;
  }
  constexpr int kStep = kThreads / kEvalDims, kFetch = kTile / kStep;
  float next[kFetch];
  const int dd = tid % kEvalDims, cc = tid / kEvalDims;
  const bool whole = t0 + kTile <= c1;
  const unsigned char *zt = (const unsigned char *)(Z + (int64_t)t0 * N);
  const uint32_t stride = (uint32_t)(kStep * N) * 4u;   // a tile's rows are within 4 MB
  auto fetch = [&](int n0) {
    const uint32_t n = n0 + dd < N ? n0 + dd : 0;
    if (whole) {
      uint32_t at = (uint32_t)(cc * N + n) * 4u;
      asm volatile("" : "+v"(at));   // the offsets are added up here, not held in registers
#pragma unroll
      for (int e = 0; e < kFetch; ++e, at += stride) next[e] = *(const float *)(zt + at);
    } else {
      uint32_t last = c1 - 1 - t0;
      asm volatile("" : "+v"(last));
#pragma unroll
      for (int e = 0; e < kFetch; ++e) {
        const uint32_t row = cc + e * kStep;
        next[e] = *(const float *)(zt + ((row < last ? row : last) * N + n) * 4u);
      }
    }
  };
  fetch(0);
  double row[kRows];
#pragma unroll
  for (int r = 0; r < kRows; ++r) row[r] = rq[r];
  for (int n0 = 0; n0 < ND; n0 += kEvalDims) {
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kFetch; ++e) stage[(cc + e * kStep) * kEvalPad + dd] = next[e];
    __syncthreads();
    if (n0 + kEvalDims < ND) {
      fetch(n0 + kEvalDims);
      if (n0 + 2 * kEvalDims > N) {   // past N: zeros, whatever stands in the row's first place
        const bool past = n0 + kEvalDims + dd >= N;
#pragma unroll
        for (int e = 0; e < kFetch; ++e) next[e] = past ? 0.f : next[e];
      }
    }
    const ScalarRows rd = rq + n0 * kRows;
    float z[kCand], zn[kCand];
#pragma unroll
    for (int c = 0; c < kCand; ++c) z[c] = stage[(c * kThreads + tid) * kEvalPad];
#pragma unroll
    for (int d = 0; d < kEvalDims; ++d) {
      // the next dimension is on its way while this one is added (the rows
      // have one dimension more than ND): its loads go behind the first use
      // of this one's, which waits for all that are out
      add(0, (double)z[0], row);
      __builtin_amdgcn_sched_barrier(0);
      double after[kRows];
#pragma unroll
      for (int r = 0; r < kRows; ++r) after[r] = rd[(d + 1) * kRows + r];
      if (d + 1 < kEvalDims)
#pragma unroll
        for (int c = 0; c < kCand; ++c) zn[c] = stage[(c * kThreads + tid) * kEvalPad + d + 1];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 1; c < kCand; ++c) add(c, (double)z[c], row);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < kRows; ++r) row[r] = after[r];
#pragma unroll
      for (int c = 0; c < kCand; ++c) z[c] = zn[c];
    }
  }
}

// One wavefront keeps the smallest pairs of a buffer of n <= 64 E: at least
// the kl smallest (all, if there are no more), at most most >= kl.  A
// distance's bits order as its value (no distance is negative), so the bound
// is found bit by bit, until the pairs below it are few enough.
template <int E>
__device__ int cut_buffer(double *bd, int32_t *bi, int n, int kl, int most, double *Td) {
  const int lane = threadIdx.x & 63;
  if (n <= kl) return n;
  unsigned long long key[E];
  int32_t id[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int p = e * 64 + lane;
    key[e] = p < n ? (unsigned long long)__double_as_longlong(bd[p]) : ~0ull;
    id[e] = p < n ? bi[p] : INT32_MAX;
  }
  unsigned long long low = 0;    // fewer than kl keys are below it
  unsigned long long top = 0;    // the bound: keys up to top, and with a key of top, ids up to itop
  int32_t itop = INT32_MAX;
  bool found = false;
  for (int b = 62; b >= 0 && !found; --b) {
    const unsigned long long mid = low | (1ull << b);
    int c = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) c += __popcll(__ballot(key[e] < mid));
    if (c < kl) {
      low = mid;
    } else if (c <= most) {
      top = mid - 1;
      found = true;
    }
  }
  if (!found) {   // ties at the kl-th distance: low is that distance, and the ids decide
    top = low;
    itop = 0;
    for (int b = 30; b >= 0; --b) {
      const int32_t mid = itop | (1 << b);
      int c = 0;
#pragma unroll
      for (int e = 0; e < E; ++e) c += __popcll(__ballot(key[e] < low || (key[e] == low && id[e] < mid)));
      if (c < kl) itop = mid;
    }
  }
  int kept = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const bool k = key[e] < top || (key[e] == top && id[e] <= itop);
    const unsigned long long m = __ballot(k);
    const int at = kept + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
    if (k) {
      bd[at] = __longlong_as_double((long long)key[e]);
      bi[at] = id[e];
    }
    kept += __popcll(m);
  }
  wave_fence();
  *Td = __longlong_as_double((long long)top);
  return kept;
}

// one wavefront sorts n pairs in place; the places up to the next power of two are filled
__device__ void sort_buffer(double *bd, int32_t *bi, int n) {
  const int lane = threadIdx.x & 63;
  int P = 64;
  while (P < n) P *= 2;
  for (int p = n + lane; p < P; p += 64) {
    bd[p] = DBL_MAX;
    bi[p] = INT32_MAX;
  }
  wave_fence();
  for (int size = 2; size <= P; size *= 2)
    for (int stride = size / 2; stride > 0; stride /= 2) {
      for (int h = lane; h < P / 2; h += 64) {
        const int i = 2 * h - (h & (stride - 1)), j = i + stride;
        const double a = bd[i], b = bd[j];
        const int32_t ia = bi[i], ib = bi[j];
        if (pair_before(b, ib, a, ia) == ((i & size) == 0) && !(a == b && ia == ib)) {
          bd[i] = b;
          bd[j] = a;
          bi[i] = ib;
          bi[j] = ia;
        }
      }
      wave_fence();
    }
}

// Neighbour lists of kl pairs of the chunk, sorted, (DBL_MAX, INT32_MAX) past
// the last.  CAP: places of a row's buffer, a tile and at least kl more.
template <bool STAGED, int DC, int CAP>
__global__ void __launch_bounds__(kThreads)
eval_near_kernel(const float *__restrict__ Z, uint32_t M, int N, int ND, const double *__restrict__ rows_d, int64_t Q,
                 int kl, uint32_t chunk, unsigned long long *row_thr, double *__restrict__ part_d,
                 int32_t *__restrict__ part_i) {
  __shared__ double bd[kRows][CAP];
  __shared__ int32_t bi[kRows][CAP];
  __shared__ double thr_d[kRows];
  __shared__ int32_t count[kRows], full[2];
  __shared__ float stage[STAGED ? kTile * kEvalPad : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t g = blockIdx.x;
  const ScalarRows rq = (ScalarRows)(rows_d + g * ND * kRows);
  const int nrows = Q - g * kRows < kRows ? (int)(Q - g * kRows) : kRows;
  if (tid < kRows) {
    thr_d[tid] = DBL_MAX;
    count[tid] = 0;
  }
  if (tid < 2) full[tid] = -1;
  __syncthreads();
  constexpr int kRoom = CAP - kThreads;            // a buffer with more than this is cut
  const int most = kl + (kRoom - kl) / 4;
  double T[kRows];
#pragma unroll
  for (int r = 0; r < kRows; ++r) T[r] = r < nrows ? DBL_MAX : -1.0;
  const uint32_t c0 = blockIdx.y * chunk, c1 = c0 + chunk < M ? c0 + chunk : M;   // below 2^32: M is below 2^31
  int step = 0;
  for (uint32_t t0 = c0; t0 < c1; t0 += kTile) {
    // the lowest threshold of the row's chunks so far
    const unsigned long long shared_thr =
        lane < nrows ? __hip_atomic_load(&row_thr[g * kRows + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    double acc[kCand][kRows];
    tile_distances<STAGED, DC>(Z, N, ND, rq, t0, c1, stage, acc);
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)shared_thr, r);
      const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(shared_thr >> 32), r);
      const double td = __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
      if (r < nrows) T[r] = td < T[r] ? td : T[r];
    }
#pragma unroll
    for (int c = 0; c < kCand; ++c, ++step) {
      const bool valid = t0 + c * kThreads + tid < c1;
      const int32_t l = (int32_t)(t0 + c * kThreads + tid);
      // lane r: the number of row r's pairs; one atomic places all rows' pairs
      int pairs = 0;
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        const int n = __popcll(__ballot(valid && acc[c][r] <= T[r]));
        pairs = lane == r ? n : pairs;
      }
      if (__ballot(pairs)) {
        int base = 0;
        if (pairs) base = atomicAdd(&count[lane], pairs);
        // full[step & 1] is written during a step, with its number, and read
        // behind its barrier; the next write to it is behind the next barrier
        if (pairs && base + pairs > kRoom) full[step & 1] = step;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
          const bool hit = valid && acc[c][r] <= T[r];
          const unsigned long long m = __ballot(hit);
          if (m == 0) continue;
          const int at = __builtin_amdgcn_readlane(base, r) +
                         __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
          if (hit) {
            bd[r][at] = acc[c][r];
            bi[r][at] = l;
          }
        }
      }
      __syncthreads();
      if (full[step & 1] != step) continue;
      for (int r = wave; r < nrows; r += kEvalWaves) {
        double td = -1.0;
        const int n = cut_buffer<CAP / 64>(bd[r], bi[r], count[r], kl, most, &td);
        if (lane == 0 && td >= 0.0) {
          count[r] = n;
          // kl pairs of lower ids are at or below td: in this chunk only what is
          // nearer follows (without this, equal points were all appended: 100,000
          // of them 2.1 ms for 1,000 rows' 10 nearest)
          thr_d[r] = td > 0.0 ? __longlong_as_double(__double_as_longlong(td) - 1) : -1.0;
          atomicMin(&row_thr[g * kRows + r], (unsigned long long)__double_as_longlong(td));
        }
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < kRows; ++r)
        if (r < nrows) T[r] = thr_d[r] < T[r] ? thr_d[r] : T[r];
    }
  }
  __syncthreads();
  for (int r = wave; r < nrows; r += kEvalWaves) {
    double td;
    const int n = cut_buffer<CAP / 64>(bd[r], bi[r], count[r], kl, most, &td);
    sort_buffer(bd[r], bi[r], n);
    const int64_t base = ((g * kRows + r) * gridDim.y + blockIdx.y) * kl;
    for (int p = lane; p < kl; p += 64) {
      part_d[base + p] = p < n ? bd[r][p] : DBL_MAX;
      part_i[base + p] = p < n ? bi[r][p] : INT32_MAX;
    }
  }
}

// best kl of the S sorted chunk lists of each row, position 0 dropped: a pair's
// place is the number of pairs before it in all lists, by binary search
__global__ void __launch_bounds__(256)
eval_merge_kernel(const double *__restrict__ part_d, const int32_t *__restrict__ part_i, int S, int kl,
                  int32_t *__restrict__ out) {
  const int64_t q = blockIdx.x;
  const double *D = part_d + q * S * kl;
  const int32_t *I = part_i + q * S * kl;
  auto before = [&](int s, double d, int32_t j) {
    int lo = 0, hi = kl;
    while (lo < hi) {
      const int mid = (lo + hi) / 2;
      if (pair_before(D[s * kl + mid], I[s * kl + mid], d, j)) lo = mid + 1;
      else hi = mid;
    }
    return lo;
  };
  for (int e = threadIdx.x; e < S * kl; e += blockDim.x) {
    const double d = D[e];
    const int32_t j = I[e];
    if (j == INT32_MAX) continue;
    int pos = 0;
    for (int s = 0; s < S && pos < kl; ++s) pos += s == e / kl ? e % kl : before(s, d, j);
    if (pos > 0 && pos < kl) out[q * (kl - 1) + pos - 1] = j;
  }
  if (threadIdx.x < kl - 1) {   // places past the last pair
    int n = 0;
    for (int s = 0; s < S && n < kl; ++s) n += before(s, DBL_MAX, INT32_MAX);
    if ((int)threadIdx.x + 1 >= n) out[q * (kl - 1) + threadIdx.x] = INT32_MAX;
  }
}

// the thresholds of rank mode, [group][kc][kRows]: the distance of each given
// candidate, in the same order of additions, and the candidate
__global__ void eval_thresholds_kernel(const float *__restrict__ Z, int N, const int32_t *__restrict__ rows, int64_t Q,
                                       const int32_t *__restrict__ cand, int kc, double *__restrict__ thr,
                                       int32_t *__restrict__ thr_j) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (Q + kRows - 1) / kRows * kRows * kc) return;
  const int64_t slot = t / kc, q = slot < Q ? slot : Q - 1;
  const int e = (int)(t - slot * kc);
  const int32_t j = cand[q * kc + e];
  const float *a = Z + (int64_t)j * N, *b = Z + (int64_t)rows[q] * N;
  double acc = 0.0;
  for (int n = 0; n < N; ++n) {
    const double d = (double)a[n] - (double)b[n];
    acc = fma(d, d, acc);
  }
  thr[((slot / kRows) * kc + e) * kRows + slot % kRows] = acc;
  thr_j[((slot / kRows) * kc + e) * kRows + slot % kRows] = j;
}

template <bool STAGED, int DC>
__global__ void __launch_bounds__(kThreads)
eval_rank_kernel(const float *__restrict__ Z, uint32_t M, int N, int ND, const double *__restrict__ rows_d, int64_t Q,
                 int kc, uint32_t chunk, const double *__restrict__ thr, const int32_t *__restrict__ thr_j,
                 int32_t *__restrict__ rank_out) {
  __shared__ float stage[STAGED ? kTile * kEvalPad : 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t g = blockIdx.x;
  const ScalarRows rq = (ScalarRows)(rows_d + g * ND * kRows);
  const uint32_t c0 = blockIdx.y * chunk, c1 = c0 + chunk < M ? c0 + chunk : M;   // below 2^32: M is below 2^31
  int32_t n[kRows];   // lane e: the count at threshold e
#pragma unroll
  for (int r = 0; r < kRows; ++r) n[r] = 0;
  for (uint32_t t0 = c0; t0 < c1; t0 += kTile) {
    double acc[kCand][kRows];
    tile_distances<STAGED, DC>(Z, N, ND, rq, t0, c1, stage, acc);
    const int32_t l0 = (int32_t)(t0 + tid);
    if (t0 + kTile > c1)   // candidates past the range are before none
#pragma unroll
      for (int c = 0; c < kCand; ++c)
#pragma unroll
        for (int r = 0; r < kRows; ++r)
          if (t0 + c * kThreads + tid >= c1) acc[c][r] = NAN;
    for (int e = 0; e < kc; ++e) {
      const ScalarRows t = (ScalarRows)(thr + (g * kc + e) * kRows);
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        const double td = t[r];
        int before = 0;
        bool tie = false;
#pragma unroll
        for (int c = 0; c < kCand; ++c) {
          before += __popcll(__ballot(acc[c][r] < td));
          tie = tie || acc[c][r] == td;
        }
        if (__ballot(tie)) {
          const int32_t j = thr_j[(g * kc + e) * kRows + r];
#pragma unroll
          for (int c = 0; c < kCand; ++c) before += __popcll(__ballot(acc[c][r] == td && l0 + c * kThreads < j));
        }
        n[r] += lane == e ? before : 0;
      }
    }
  }
  if (lane < kc)
#pragma unroll
    for (int r = 0; r < kRows; ++r)
      if (g * kRows + r < Q && n[r]) atomicAdd(&rank_out[(g * kRows + r) * kc + lane], n[r]);
}

// per-row counts of the sample scores, summed with integer atomics (exact,
// order-free): [0] |v ∩ n| over the first k, [1] same-label neighbours in n,
// [2] sum over n \ v of (rank in X - k)
__global__ void eval_scores_kernel(const int32_t *__restrict__ rows, int64_t Q, const int32_t *__restrict__ nx, int kx,
                                   const int32_t *__restrict__ ny, int ky, const int32_t *__restrict__ rank_y,
                                   const int32_t *__restrict__ labels, int k, unsigned long long *__restrict__ sums) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= Q) return;
  unsigned long long hits = 0, same = 0, trust = 0;
  const int32_t *vx = nx ? nx + q * kx : nullptr;
  const int32_t *vy = ny + q * ky;
  const int32_t lab = labels ? labels[rows[q]] : 0;
  for (int c = 0; c < k; ++c) {
    const int32_t j = vy[c];
    bool in_x = false;
    if (vx)
      for (int e = 0; e < k; ++e) in_x = in_x || vx[e] == j;
    hits += in_x ? 1 : 0;
    if (labels) same += labels[j] == lab ? 1 : 0;
    if (rank_y && !in_x) trust += (unsigned long long)(rank_y[q * ky + c] - k);
  }
  atomicAdd(&sums[0], hits);
  atomicAdd(&sums[1], same);
  atomicAdd(&sums[2], trust);
}

__global__ void eval_zero_kernel(int32_t *p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// Chunks of the candidate range: blocks for some four rounds of the chip, so
// that the last, partly filled round weighs little, in chunks of at least 2048
// candidates (a chunk's first tiles all pass the thresholds); at most 64.
int eval_chunks(int64_t Q, int64_t M) {
  const int64_t groups = (Q + kRows - 1) / kRows;
  int64_t S = (2048 + groups - 1) / groups;
  const int64_t smax = M / 2048 > 1 ? M / 2048 : 1;
  if (S > smax) S = smax;
  if (S > 64) S = 64;
  return (int)S;
}

int eval_dims(int N) { return N <= 2 ? 2 : N <= 4 ? 4 : N <= 8 ? 8 : (N + kEvalDims - 1) / kEvalDims * kEvalDims; }

// rows taken at a time (a multiple of kRows) at so many bytes of scratch each
int64_t eval_band(int64_t Q, int64_t row_bytes) {
  int64_t band = kEvalRowBytes / row_bytes / kRows * kRows;
  if (band < 64 * kRows) band = 64 * kRows;
  return band < Q ? band : Q;
}

struct EvalScratch {
  int64_t band = 0;   // rows taken at a time
  int S = 1;
  double *rq = nullptr, *part_d = nullptr, *thr = nullptr;
  unsigned long long *row_thr = nullptr;
  int32_t *part_i = nullptr, *thr_j = nullptr;
};

template <bool STAGED, int DC>
void near_dc(dim3 grid, const float *Z, uint32_t M, int N, const double *rq, int64_t Q, int kl, uint32_t chunk,
             const EvalScratch &w, hipStream_t s) {
  // 320 places (three blocks to a CU above 8 dimensions, against two) while a cut leaves half the room free
  if (kl <= 32)
    eval_near_kernel<STAGED, DC, 320><<<grid, kThreads, 0, s>>>(Z, M, N, eval_dims(N), rq, Q, kl, chunk, w.row_thr, w.part_d,
                                                               w.part_i);
  else
    eval_near_kernel<STAGED, DC, 512><<<grid, kThreads, 0, s>>>(Z, M, N, eval_dims(N), rq, Q, kl, chunk, w.row_thr, w.part_d,
                                                               w.part_i);
}

int eval_max_k() { return 128; }
int eval_max_rank_k() { return 64; }
int eval_max_dims() { return 1024; }

void launch_rows(const float *Z, int N, const int32_t *rows, int64_t Q, const EvalScratch &w, hipStream_t s) {
  const int ND = eval_dims(N);
  eval_rows_kernel<<<grid_for((Q + kRows - 1) / kRows * kRows * ND), kBlock, 0, s>>>(Z, N, ND, rows, Q, w.rq,
                                                                                           w.row_thr);
}

hipError_t launch_eval_neighbours(const float *Z, int64_t M, int N, const int32_t *rows, int64_t Q, int k,
                                  const EvalScratch &w, int32_t *out, hipStream_t s) {
  const int kl = k + 1;
  const uint32_t chunk = (uint32_t)((M + w.S - 1) / w.S);
  for (int64_t q0 = 0; q0 < Q; q0 += w.band) {
    const int64_t n = Q - q0 < w.band ? Q - q0 : w.band;
    const dim3 grid((unsigned)((n + kRows - 1) / kRows), (unsigned)w.S);
    launch_rows(Z, N, rows + q0, n, w, s);
    auto near = N <= 2 ? near_dc<false, 2> : N <= 4 ? near_dc<false, 4> : N <= 8 ? near_dc<false, 8> : near_dc<true, 0>;
    near(grid, Z, (uint32_t)M, N, w.rq, n, kl, chunk, w, s);
    eval_merge_kernel<<<(unsigned)n, 256, 0, s>>>(w.part_d, w.part_i, w.S, kl, out + q0 * k);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_eval_ranks(const float *Z, int64_t M, int N, const int32_t *rows, int64_t Q, const int32_t *cand,
                             int kc, const EvalScratch &w, int32_t *rank_out, hipStream_t s) {
  const uint32_t chunk = (uint32_t)((M + w.S - 1) / w.S);
  const int ND = eval_dims(N);
  eval_zero_kernel<<<grid_for(Q * kc), kBlock, 0, s>>>(rank_out, Q * kc);
  for (int64_t q0 = 0; q0 < Q; q0 += w.band) {
    const int64_t n = Q - q0 < w.band ? Q - q0 : w.band;
    const dim3 grid((unsigned)((n + kRows - 1) / kRows), (unsigned)w.S);
    launch_rows(Z, N, rows + q0, n, w, s);
    eval_thresholds_kernel<<<grid_for((n + kRows - 1) / kRows * kRows * kc), kBlock, 0, s>>>(
        Z, N, rows + q0, n, cand + q0 * kc, kc, w.thr, w.thr_j);
    auto scan = N <= 2   ? eval_rank_kernel<false, 2>
                : N <= 4 ? eval_rank_kernel<false, 4>
                : N <= 8 ? eval_rank_kernel<false, 8>
                         : eval_rank_kernel<true, 0>;
    scan<<<grid, kThreads, 0, s>>>(Z, (uint32_t)M, N, ND, w.rq, n, kc, chunk, w.thr, w.thr_j, rank_out + q0 * kc);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_eval_scores(const int32_t *rows, int64_t Q, const int32_t *nx, int kx, const int32_t *ny, int ky,
                              const int32_t *rank_y, const int32_t *labels, int k, unsigned long long *sums,
                              hipStream_t s) {
  eval_zero_kernel<<<1, kBlock, 0, s>>>((int32_t *)sums, 6);
  eval_scores_kernel<<<grid_for(Q), kBlock, 0, s>>>(rows, Q, nx, kx, ny, ky, rank_y, labels, k, sums);
  return hipGetLastError();
}

}  // namespace
}  // namespace ivhd

// ---- C ABI ----------------------------------------------------------------
using namespace ivhd;

namespace {

int check_sample(const float *d_z, int64_t M, int32_t N, const int32_t *d_rows, int64_t Q) {
  if (!d_z || (Q > 0 && !d_rows)) return fail(IVHD_EINVAL, "d_z and d_rows must not be NULL");
  if (M < 2 || M > (int64_t)INT32_MAX - 1) return fail(IVHD_EINVAL, "M = %lld outside [2, 2^31-2]", (long long)M);
  if (N < 1 || N > eval_max_dims()) return fail(IVHD_EINVAL, "N = %d outside [1, %d]", N, eval_max_dims());
  if (Q < 0) return fail(IVHD_EINVAL, "Q = %lld < 0", (long long)Q);
  return IVHD_OK;
}

// device range check of index arrays (entries must lie in [0, hi)); synchronises s
int check_indices(const int32_t *const *arrays, const int64_t *counts, int n, int64_t hi, hipStream_t s) {
  int32_t *flags = nullptr;
  int rc = dev_alloc(&flags, FLAG_SLOTS, "device flags");
  if (rc) return rc;
  hipError_t e = launch_fill_i32(flags, FLAG_SLOTS, 0, s);
  for (int a = 0; a < n && e == hipSuccess; ++a)
    if (arrays[a] && counts[a] > 0) e = launch_range_check(arrays[a], counts[a], (int32_t)hi, flags, s);
  int32_t h[FLAG_SLOTS] = {0};
  if (e == hipSuccess) e = hipMemcpyAsync(h, flags, sizeof h, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  dev_free(flags, s);
  if (e != hipSuccess) return hip_fail(e, "index range check");
  if (h[FLAG_BAD_INDEX]) return fail(IVHD_EINVAL, "an index entry is outside [0, %lld)", (long long)hi);
  return IVHD_OK;
}

}  // namespace

extern "C" {

int ivhd_eval_neighbours(const float *d_z, int64_t M, int32_t N, const int32_t *d_rows, int64_t Q, int32_t k,
                         int32_t *d_idx, void *stream) {
  clear_error();
  int rc = check_sample(d_z, M, N, d_rows, Q);
  if (rc) return rc;
  if (!d_idx) return fail(IVHD_EINVAL, "d_idx is NULL");
  const int64_t kmax = M - 1 < eval_max_k() ? M - 1 : eval_max_k();
  if (k < 1 || k > kmax) return fail(IVHD_EINVAL, "k = %d outside [1, %lld]", k, (long long)kmax);
  if (Q == 0) return IVHD_OK;
  hipStream_t s = (hipStream_t)stream;
  const int32_t *arrays[] = {d_rows};
  const int64_t counts[] = {Q};
  if ((rc = check_indices(arrays, counts, 1, M, s))) return rc;
  EvalScratch w;
  w.S = eval_chunks(Q, M);
  const int64_t list = (int64_t)w.S * (k + 1), nd = eval_dims(N);
  w.band = eval_band(Q, nd * 8 + 8 + list * 12);
  const int64_t slots = (w.band + kRows - 1) / kRows * kRows;
  Scratch S(s);
  Carve c;
  c.add(&w.rq, (size_t)(slots * nd + kRows));   // the scan loads a dimension ahead
  c.add(&w.row_thr, (size_t)w.band);
  c.add(&w.part_d, (size_t)(w.band * list));
  c.add(&w.part_i, (size_t)(w.band * list));
  if ((rc = c.get(S, "sample rows and chunk lists"))) return rc;
  hipError_t e = launch_eval_neighbours(d_z, M, N, d_rows, Q, k, w, d_idx, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e, "eval neighbours");
  return IVHD_OK;
}

int ivhd_eval_ranks(const float *d_z, int64_t M, int32_t N, const int32_t *d_rows, int64_t Q, const int32_t *d_cand,
                    int32_t kc, int32_t *d_rank, void *stream) {
  clear_error();
  int rc = check_sample(d_z, M, N, d_rows, Q);
  if (rc) return rc;
  if (!d_cand || !d_rank) return fail(IVHD_EINVAL, "d_cand and d_rank must not be NULL");
  if (kc < 1 || kc > eval_max_rank_k()) return fail(IVHD_EINVAL, "kc = %d outside [1, %d]", kc, eval_max_rank_k());
  if (Q == 0) return IVHD_OK;
  hipStream_t s = (hipStream_t)stream;
  const int32_t *arrays[] = {d_rows, d_cand};
  const int64_t counts[] = {Q, Q * kc};
  if ((rc = check_indices(arrays, counts, 2, M, s))) return rc;
  EvalScratch w;
  w.S = eval_chunks(Q, M);
  const int64_t nd = eval_dims(N);
  w.band = eval_band(Q, nd * 8 + kc * 12);
  const int64_t slots = (w.band + kRows - 1) / kRows * kRows;
  Scratch S(s);
  Carve c;
  c.add(&w.rq, (size_t)(slots * nd + kRows));
  c.add(&w.thr, (size_t)(slots * kc));
  c.add(&w.thr_j, (size_t)(slots * kc));
  if ((rc = c.get(S, "sample rows and thresholds"))) return rc;
  hipError_t e = launch_eval_ranks(d_z, M, N, d_rows, Q, d_cand, kc, w, d_rank, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e, "eval ranks");
  return IVHD_OK;
}

int ivhd_eval_scores(int64_t M, const int32_t *d_rows, int64_t Q, const int32_t *d_nx, int32_t kx, const int32_t *d_ny,
                     int32_t ky, const int32_t *d_rank_y, const int32_t *d_labels, int32_t k, double *h_out,
                     void *stream) {
  clear_error();
  if (!h_out) return fail(IVHD_EINVAL, "h_out is NULL");
  if (!d_ny || !d_rows) return fail(IVHD_EINVAL, "d_rows and d_ny must not be NULL");
  if (M < 2 || M > (int64_t)INT32_MAX - 1) return fail(IVHD_EINVAL, "M = %lld outside [2, 2^31-2]", (long long)M);
  if (Q < 1) return fail(IVHD_EINVAL, "Q = %lld < 1", (long long)Q);
  if (k < 1 || k > ky) return fail(IVHD_EINVAL, "k = %d outside [1, ky = %d]", k, ky);
  if (d_nx && k > kx) return fail(IVHD_EINVAL, "k = %d above kx = %d", k, kx);
  if (d_rank_y && !d_nx) return fail(IVHD_EINVAL, "d_rank_y needs d_nx (the ranks count only points outside it)");
  hipStream_t s = (hipStream_t)stream;
  const int32_t *arrays[] = {d_rows, d_ny, d_nx};
  const int64_t counts[] = {Q, Q * ky, d_nx ? Q * kx : 0};
  int rc = check_indices(arrays, counts, 3, M, s);
  if (rc) return rc;
  unsigned long long *sums = nullptr;
  if ((rc = dev_alloc(&sums, 3, "score sums"))) return rc;
  unsigned long long h[3] = {0, 0, 0};
  hipError_t e = launch_eval_scores(d_rows, Q, d_nx, kx, d_ny, ky, d_rank_y, d_labels, k, sums, s);
  if (e == hipSuccess) e = hipMemcpyAsync(h, sums, sizeof h, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  dev_free(sums, s);
  if (e != hipSuccess) return hip_fail(e, "eval scores");
  const double kq = (double)k * (double)Q;
  h_out[0] = d_nx ? (double)h[0] / kq : NAN;
  h_out[1] = d_labels ? (double)h[1] / kq : NAN;
  const double den = kq * (2.0 * (double)M - 3.0 * k - 1.0);
  h_out[2] = (d_rank_y && den > 0) ? 1.0 - 2.0 / den * (double)h[2] : NAN;
  return IVHD_OK;
}

}  // extern "C"
