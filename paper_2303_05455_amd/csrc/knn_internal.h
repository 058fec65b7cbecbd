// Declarations of the kNN search (knn_filter.hip) and the scratch buffers of
// the stateless calls.  Not part of the public ABI.
#pragma once

#include <new>
#include <vector>

#include "ivhd_internal.h"

namespace ivhd {

// device buffers of work on one stream, released together
struct Scratch {
  std::vector<void *> bufs;
  hipStream_t stream;
  explicit Scratch(hipStream_t s = nullptr) : stream(s) {}
  Scratch(const Scratch &) = delete;
  Scratch &operator=(const Scratch &) = delete;
  ~Scratch() { dev_free_all(bufs.data(), bufs.size(), stream); }
  template <typename T>
  int get(T **p, size_t n, const char *what) {
    *p = nullptr;
    try {   // room for it first: nothing is thrown across the ABI
      bufs.reserve(bufs.size() + 1);
    } catch (const std::bad_alloc &) {
      return fail(IVHD_ENOMEM, "host memory for the buffer list (%s)", what);
    }
    int rc = dev_alloc(p, n, what);
    if (!rc) bufs.push_back(*p);
    return rc;
  }
};

// several buffers out of one allocation (each on a 256-byte boundary)
struct Carve {
  static constexpr int kMost = 16;
  struct Part {
    void **p;
    size_t at;
  } parts[kMost];
  int n_parts = 0;
  size_t bytes = 0;
  template <typename T>
  void add(T **p, size_t n) {
    if (n_parts < kMost) parts[n_parts] = {reinterpret_cast<void **>(p), bytes};
    ++n_parts;
    bytes += (n * sizeof(T) + 255) / 256 * 256;
  }
  int get(Scratch &S, const char *what) {
    if (n_parts > kMost) return fail(IVHD_ESTATE, "%d buffers in one allocation (%s)", n_parts, what);
    unsigned char *base;
    const int rc = S.get(&base, bytes, what);
    if (!rc)
      for (int i = 0; i < n_parts; ++i) *parts[i].p = base + parts[i].at;
    return rc;
  }
};

// What a set of rows has at most, as float bits (non-negative floats compare as
// integers; zero before use): the squared norm, and for each class of squared
// norms (by their exponents) the squared rounding residual of a row, in the end
// the residual of a row up to that class
constexpr int kNormClasses = 256;
struct KnnStats {
  uint32_t norm2, res[kNormClasses];
};
// operand images of whole tiles of rows, and the room that was allocated
struct KnnImage {
  _Float16 *p = nullptr;
  int64_t halves = 0;
};
// One search: k nearest of M candidate rows to each of nq rows of Q (same: the
// candidates are Q).  What open allocates lives as long as it does and is never
// replaced; what a run needs beyond that, for the queries that it repeats, is
// the run's own.
struct KnnSearch {
  // allocates, and takes the centre and the scale of all operands from a sample
  // of the rows `sample` (IVHD_EINVAL when they or Q are not finite).  Synchronises.
  int open(int64_t M, int N, const float *Q, int64_t nq, const float *sample, int64_t sample_rows, bool same, int k,
           hipStream_t s);
  // the answers for the candidates X [M][N]; self_mode: 0 = none, 1 = query q
  // excludes candidate q, 2 = query q excludes self[q].  Synchronises the
  // stream.  It may be called again with as many other candidates and the same
  // queries, which are prepared once.
  int run(const float *X, int self_mode, const int32_t *self, int32_t *idx, float *dist);
  // the answers of queries rows[0..n) (NULL: all) from all exact distances
  int rank_all(const float *X, const int32_t *rows, int64_t n, int self_mode, const int32_t *self, int32_t *idx,
               float *dist);

  Scratch S;
  int64_t M = 0, nq = 0;
  int N = 0, k = 0;
  const float *Q = nullptr;
  bool same = false, few = false, direct = false, queries_ready = false;
  float scale = 1.f;
  hipStream_t s = nullptr;
  KnnImage ch, cl, qh, ql;   // operands, high and low; the low ones only with few
  float *start = nullptr, *qnorm = nullptr, *qres = nullptr, *mean = nullptr;
  KnnStats *xstats = nullptr;
  float *fail_dist = nullptr;
  int32_t *fails = nullptr, *pilot = nullptr, *order = nullptr;
  int64_t place_of = 1;
  uint64_t *part = nullptr;
  int64_t part_cap = 0;
};

}  // namespace ivhd
