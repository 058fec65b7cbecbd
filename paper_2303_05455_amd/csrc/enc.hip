// Kernels of the parametric encoder (an MLP N-D -> 2-D trained on the IVHD
// stress): BF16 operands on the gfx950 matrix cores with FP32 accumulation.
//
// gemm_bf16: C[M][N] = sum_k opA[m][k] opB[k][n]
//   opA[m][k] = A[m*lda + k]  (ta = 0)  or  A[k*lda + m]  (ta = 1)
//   opB[k][n] = B[k*ldb + n]  (tb = 0)  or  B[n*ldb + k]  (tb = 1)
// Waves own 64 x 64 output blocks; operands are staged in LDS with K
// contiguous per row, so one lane's MFMA operand (8 consecutive k) is a
// single 16-byte LDS read.  The instruction is v_mfma_f32_16x16x32_bf16:
// lane l supplies A[l%16][8(l/16)..+8) and B[8(l/16)..+8)[l%16], and
// receives D[4(l/16)+r][l%16], r = 0..3.
// Three kernels: gemm_nt_kernel when both operands are K-contiguous (ta = 0,
// tb = 1) with 16-byte rows, gemm_tn_kernel when both are K-major (ta = 1,
// tb = 0) with 16-byte rows: the training step's input and weight gradients,
// 256 x 128 tiles of 8 waves, K steps of 32 through a ring of LDS stages filled
// by direct-to-LDS loads; gemm_kernel for every other layout: 128 x 128 tiles
// of 4 waves, K steps of 32 staged through registers.
// Epilogues: FP32 store (split-K partials: the K split selects the K range
// and the output slab), bias + ReLU -> BF16, or (dgrad) multiply by the
// ReLU derivative read from the forward activation -> BF16.
//
// Rounding: every FP32 -> BF16 conversion is round-to-nearest-even.
#include "enc_internal.h"

namespace ivhd {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int TM = 128, TN = 128, TK = 32;
constexpr int KP = TK + 8;   // LDS row pitch in bf16 (80 bytes: 16-byte aligned rows)
constexpr int kGemmThreads = 256;
constexpr int kColsumLanes = 8, kColsumThreads = 32 * kColsumLanes;   // row lanes of the column sums

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// to nearest even, a NaN quietened: the conversion instruction's results, which
// the eight integer operations of doing it by hand have for every float
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

struct alignas(16) U16x8 {
  uint16_t v[8];
};

struct alignas(8) U16x4 {
  uint16_t v[4];
};

// one operand tile (rows r0..r0+127 of op, k0..k0+31) in two halves, so the
// global loads of step s + 1 can be issued before the MFMAs of step s:
// op[row][k] = T ? P[k*ld + row] : P[row*ld + k]; out of range -> 0.
// Each thread holds two 8-element chunks.
struct TileFrag {
  U16x8 v[2];
};

template <bool T>
__device__ __forceinline__ void load_tile(TileFrag &F, const uint16_t *__restrict__ P, int64_t ld, int64_t rows,
                                          int64_t r0, int64_t k0, int64_t kend, bool vec_ok) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int id = tid + kGemmThreads * c;
    U16x8 &v = F.v[c];
    if (!T) {
      // 128 rows x 4 chunks of 8 k
      const int r = id >> 2, kc = (id & 3) * 8;
      const int64_t row = r0 + r, k = k0 + kc;
      if (row < rows && vec_ok && k + 8 <= kend) {
        v = *reinterpret_cast<const U16x8 *>(P + row * ld + k);
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) v.v[j] = (row < rows && k + j < kend) ? P[row * ld + k + j] : (uint16_t)0;
      }
    } else {
      // k-major source: 32 k x 16 chunks of 8 rows
      const int kk = id >> 4, rc = (id & 15) * 8;
      const int64_t k = k0 + kk, row = r0 + rc;
      if (k < kend && vec_ok && row + 8 <= rows) {
        v = *reinterpret_cast<const U16x8 *>(P + k * ld + row);
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) v.v[j] = (k < kend && row + j < rows) ? P[k * ld + row + j] : (uint16_t)0;
      }
    }
  }
}

template <bool T>
__device__ __forceinline__ void store_tile(const TileFrag &F, uint16_t *__restrict__ lds) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int id = tid + kGemmThreads * c;
    if (!T) {
      const int r = id >> 2, kc = (id & 3) * 8;
      *reinterpret_cast<U16x8 *>(lds + r * KP + kc) = F.v[c];
    } else {
      const int kk = id >> 4, rc = (id & 15) * 8;
#pragma unroll
      for (int j = 0; j < 8; ++j) lds[(rc + j) * KP + kk] = F.v[c].v[j];
    }
  }
}

// Epilogue of a 128 x 128 tile: wave (wm, wn) holds rows wm..wm+63 and
// columns wn..wn+63 as 4 x 4 MFMA results; lane l has column l%16 and rows
// 4(l/16)..+4 of each.  z selects the FP32 split-K slab.
template <int EPI>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs &g, const floatx4 (&acc)[4][4], int64_t m0, int64_t n0,
                                              int wm, int wn, int lane, int64_t z) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t n = n0 + wn + 16 * j + (lane & 15);
      if (n >= g.N) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t m = m0 + wm + 16 * i + 4 * (lane >> 4) + r;
        if (m >= g.M) continue;
        float x = acc[i][j][r];
        if (EPI == GEMM_EPI_F32) {
          float *C = static_cast<float *>(g.C) + z * g.M * g.ldc;
          C[m * g.ldc + n] = x;
        } else if (EPI == GEMM_EPI_BIAS_RELU_BF16) {
          x += g.bias ? g.bias[n] : 0.f;
          x = fmaxf(x, 0.f);
          static_cast<uint16_t *>(g.C)[m * g.ldc + n] = f2bf(x);
        } else {   // GEMM_EPI_RELU_MASK_BF16
          const float h = bf2f(g.mask[m * g.ldm + n]);
          static_cast<uint16_t *>(g.C)[m * g.ldc + n] = f2bf(h > 0.f ? x : 0.f);
        }
      }
    }
  }
}

template <bool TA, bool TB, int EPI>
__global__ void __launch_bounds__(kGemmThreads) gemm_kernel(GemmArgs g) {
  __shared__ __attribute__((aligned(16))) uint16_t As[TM * KP];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[TN * KP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t m0 = (int64_t)blockIdx.y * TM, n0 = (int64_t)blockIdx.x * TN;
  const int64_t kbeg = (int64_t)blockIdx.z * g.kchunk;
  const int64_t kend = kbeg + g.kchunk < g.K ? kbeg + g.kchunk : g.K;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;

  floatx4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // A rows are m: opA[m][k] is P[row*ld + k] unless transposed.  B rows are
  // n: opB[k][n] is P[row*ld + k] exactly when B is given transposed.
  TileFrag fa, fb;
  load_tile<TA>(fa, g.A, g.lda, g.M, m0, kbeg, kend, g.vec_a);
  load_tile<!TB>(fb, g.B, g.ldb, g.N, n0, kbeg, kend, g.vec_b);
  for (int64_t k0 = kbeg; k0 < kend; k0 += TK) {
    __syncthreads();
    store_tile<TA>(fa, As);
    store_tile<!TB>(fb, Bs);
    __syncthreads();
    if (k0 + TK < kend) {   // the next step's loads fly during this step's MFMAs
      load_tile<TA>(fa, g.A, g.lda, g.M, m0, k0 + TK, kend, g.vec_a);
      load_tile<!TB>(fb, g.B, g.ldb, g.N, n0, k0 + TK, kend, g.vec_b);
    }
    const int kq = (lane >> 4) * 8;
    bf16x8 a[4], b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      a[i] = *reinterpret_cast<const bf16x8 *>(As + (wm + 16 * i + (lane & 15)) * KP + kq);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      b[j] = *reinterpret_cast<const bf16x8 *>(Bs + (wn + 16 * j + (lane & 15)) * KP + kq);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
  }

  gemm_epilogue<EPI>(g, acc, m0, n0, wm, wn, lane, blockIdx.z);
}

// ---- both operands K-contiguous (opA = A[m][k], opB = B[n][k]) -----------
// Tiles of 256 x 128 per block of 512 threads (8 waves of 64 x 64, four
// along M by two along N).  K goes in steps of 32 through a ring of three
// LDS stages that global_load_lds_dwordx4 fills directly (no register
// staging): a step's loads are issued two steps ahead, each wave waits for
// its own loads of the step with vmcnt, and one barrier per step publishes
// the stage and frees the one loaded next.  A stage holds the A rows then
// the B rows, 64 bytes each (four 16-byte chunks of k); the load writes lane
// l's chunk at stage slot base + l, so each lane picks which chunk to fetch,
// and chunk c of row r sits in slot 4 r + (c ^ ((r >> 1) & 3)): the 16 rows
// an MFMA operand read touches then fall on distinct bank groups.  Two
// blocks share a CU (74 KB of LDS each), so one block's epilogue overlaps
// the other's loop.  Tiles are dealt to the XCDs in contiguous runs (blocks
// go to XCD b % 8), ordered by K split, then along the longer output side,
// then the shorter one: the tiles that share a panel of the long operand,
// and the tiles of one K split, run on one XCD and share its L2.  Requires
// 16-byte aligned operands with lda, ldb and K multiples of 8, so every
// chunk is wholly inside or outside the matrix: a chunk past the last row
// reads the operand's first chunk instead (its outputs are never stored),
// and chunks past the end of K are zeroed in LDS once they have arrived.
// Measured at 57,344 x 784 x 512: 74.6 us against 96.7 us for 128 x 128
// tiles with register staging.
constexpr int NTK = 64;        // K granularity of a split-K chunk
constexpr int kXcds = 8;
constexpr int BM = 256, BN = 128, BK = 32;
constexpr int kNtThreads = 512;
constexpr int kRing = 3;
constexpr int kStage = (BM + BN) * BK;            // bf16 per stage
constexpr int kStageLoads = (BM + BN) * BK / 8 / kNtThreads;   // 16-byte chunks per thread per stage
static_assert(kStageLoads * kNtThreads * 8 == kStage, "a stage is a whole number of wave loads");
constexpr int kCbPitch = BN + 8;                 // bf16 epilogue tile pitch (272 bytes)
constexpr int kCfPitch = BN + 4;                 // FP32 epilogue half-tile pitch
static_assert(BM * kCbPitch * 2 <= kRing * kStage * 2, "bf16 tile must fit in the ring");
static_assert(BM / 2 * kCfPitch * 4 <= kRing * kStage * 2, "FP32 half tile must fit in the ring");

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ int ring_slot(int row, int chunk) { return row * 4 + (chunk ^ ((row >> 1) & 3)); }

// Epilogue of both 256 x 128 kernels; the ring S is free.
template <int EPI>
__device__ __forceinline__ void ring_epilogue(const GemmArgs &g, const floatx4 (&acc)[4][4], uint16_t *S, int64_t m0,
                                              int64_t n0, int64_t z) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  // Epilogue.  Wave (wm, wn) holds rows wm..wm+63 and columns wn..wn+63 as
  // 4 x 4 MFMA results; lane l has column l % 16 and rows 4 (l / 16)..+4 of
  // each.  The tile goes through LDS so that every thread finishes whole row
  // chunks with 16-byte stores where the leading dimension and pointer allow.
  if (EPI == GEMM_EPI_F32) {
    // FP32 in two halves of 128 rows (waves 0-3, then 4-7)
    float *Cf = reinterpret_cast<float *>(S);
    float *C = static_cast<float *>(g.C) + z * g.M * g.ldc;
    const bool vec = g.ldc % 4 == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if ((wave >> 2) == half) {
#pragma unroll
        for (int ii = 0; ii < 4; ++ii)
#pragma unroll
          for (int jj = 0; jj < 4; ++jj)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              Cf[(wm - 128 * half + 16 * ii + 4 * (lane >> 4) + r) * kCfPitch + wn + 16 * jj + (lane & 15)] =
                  acc[ii][jj][r];
      }
      __syncthreads();
#pragma unroll
      for (int c = 0; c < 8; ++c) {   // 128 rows x 32 chunks of 4
        const int id = tid + kNtThreads * c, m = id >> 5, qc = (id & 31) * 4;
        const int64_t row = m0 + 128 * half + m, col = n0 + qc;
        if (row >= g.M || col >= g.N) continue;
        const floatx4 v = *reinterpret_cast<const floatx4 *>(Cf + m * kCfPitch + qc);
        if (vec && col + 4 <= g.N) {
          *reinterpret_cast<floatx4 *>(C + row * g.ldc + col) = v;
        } else {
          for (int e = 0; e < 4 && col + e < g.N; ++e) C[row * g.ldc + col + e] = v[e];
        }
      }
      __syncthreads();
    }
    return;
  }
  // BF16 outputs: bias + ReLU applied in FP32 before rounding; the ReLU mask
  // (a zero or a copy of the rounded value) after it, which is the same
  uint16_t *Cb = S;
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    const int64_t col = n0 + wn + 16 * jj + (lane & 15);
    const float bv = EPI == GEMM_EPI_BIAS_RELU_BF16 && g.bias && col < g.N ? g.bias[col] : 0.f;
#pragma unroll
    for (int ii = 0; ii < 4; ++ii)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float v = acc[ii][jj][r];
        if (EPI == GEMM_EPI_BIAS_RELU_BF16) v = fmaxf(v + bv, 0.f);
        Cb[(wm + 16 * ii + 4 * (lane >> 4) + r) * kCbPitch + wn + 16 * jj + (lane & 15)] = f2bf(v);
      }
  }
  __syncthreads();
  uint16_t *C = static_cast<uint16_t *>(g.C);
  const bool vec = g.ldc % 8 == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0;
  const bool vec_m = EPI == GEMM_EPI_RELU_MASK_BF16 && g.ldm % 8 == 0 &&
                     (reinterpret_cast<uintptr_t>(g.mask) & 15) == 0;
  // 256 rows x 16 chunks of 8: thread chunk c is row (tid >> 4) + 32 c.
  // Whole mask chunks are loaded first, branch-free (others read the first
  // chunk and are replaced element by element below).
  U16x8 mk[8];
  if (EPI == GEMM_EPI_RELU_MASK_BF16) {
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int64_t row = m0 + (tid >> 4) + 32 * c, col = n0 + (tid & 15) * 8;
      const bool full = vec_m && row < g.M && col + 8 <= g.N;
      mk[c] = *reinterpret_cast<const U16x8 *>(full ? g.mask + row * g.ldm + col : g.mask);
    }
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int m = (tid >> 4) + 32 * c, qc = (tid & 15) * 8;
    const int64_t row = m0 + m, col = n0 + qc;
    if (row >= g.M || col >= g.N) continue;
    U16x8 o = *reinterpret_cast<const U16x8 *>(Cb + m * kCbPitch + qc);
    if (EPI == GEMM_EPI_RELU_MASK_BF16) {
      if (!(vec_m && col + 8 <= g.N))
        for (int e = 0; e < 8; ++e) mk[c].v[e] = col + e < g.N ? g.mask[row * g.ldm + col + e] : (uint16_t)0;
#pragma unroll
      for (int e = 0; e < 8; ++e) o.v[e] = bf2f(mk[c].v[e]) > 0.f ? o.v[e] : (uint16_t)0;
    }
    if (vec && col + 8 <= g.N) {
      *reinterpret_cast<U16x8 *>(C + row * g.ldc + col) = o;
    } else {
      for (int e = 0; e < 8 && col + e < g.N; ++e) C[row * g.ldc + col + e] = o.v[e];
    }
  }
}

template <int EPI>
__global__ void __launch_bounds__(kNtThreads, 2) gemm_nt_kernel(GemmArgs g, int64_t tiles_m, int64_t tiles_n) {
  __shared__ __attribute__((aligned(16))) uint16_t S[kRing * kStage];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t nb = (int64_t)gridDim.x, lin = blockIdx.x;
  const int64_t q = nb / kXcds, rem = nb % kXcds, x = lin % kXcds, i = lin / kXcds;
  const int64_t tile = x < rem ? x * (q + 1) + i : rem * (q + 1) + (x - rem) * q + i;
  const int64_t per_z = tiles_m * tiles_n, z = tile / per_z, t = tile % per_z;
  const bool m_outer = tiles_m >= tiles_n;
  const int64_t m0 = (m_outer ? t / tiles_n : t % tiles_m) * BM;
  const int64_t n0 = (m_outer ? t % tiles_n : t / tiles_m) * BN;
  const int64_t kbeg = z * g.kchunk;
  const int64_t kend = kbeg + g.kchunk < g.K ? kbeg + g.kchunk : g.K;
  const int nsteps = (int)((kend - kbeg + BK - 1) / BK);
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;

  // this thread's chunks of every stage: slot (wave * kStageLoads + c) * 64 + lane
  int row_of[kStageLoads], chunk_of[kStageLoads];
#pragma unroll
  for (int c = 0; c < kStageLoads; ++c) {
    const int slot = (wave * kStageLoads + c) * 64 + lane, r = slot >> 2;
    row_of[c] = r;
    chunk_of[c] = (slot & 3) ^ ((r >> 1) & 3);
  }
  auto issue = [&](int st) {
    const int64_t k0 = kbeg + (int64_t)st * BK;
    uint16_t *base = S + (st % kRing) * kStage;
#pragma unroll
    for (int c = 0; c < kStageLoads; ++c) {
      const int64_t k = k0 + chunk_of[c] * 8;
      const int r = row_of[c];
      const uint16_t *p;
      if (r < BM) {
        const int64_t ra = m0 + r;
        p = ra < g.M && k < kend ? g.A + ra * g.lda + k : g.A;
      } else {
        const int64_t rb = n0 + (r - BM);
        p = rb < g.N && k < kend ? g.B + rb * g.ldb + k : g.B;
      }
      __builtin_amdgcn_global_load_lds((const void *)p, (lds_void *)(base + (wave * kStageLoads + c) * 64 * 8), 16,
                                       0, 0);
    }
  };

  floatx4 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};

  static_assert(kRing == 3 && kStageLoads == 3, "the vmcnt waits below count three loads per stage");
  int issued = 0;
  for (; issued < kRing - 1 && issued < nsteps; ++issued) issue(issued);
  for (int st = 0; st < nsteps; ++st) {
    // this step's loads are done once at most the later stages' remain
    if (issued - st - 1 >= 1) asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    uint16_t *base = S + (st % kRing) * kStage;
    if (kbeg + (int64_t)(st + 1) * BK > kend) {   // K tail: zero this thread's chunks past the end
#pragma unroll
      for (int c = 0; c < kStageLoads; ++c)
        if (kbeg + (int64_t)st * BK + chunk_of[c] * 8 >= kend)
          *reinterpret_cast<u32x4 *>(base + (wave * kStageLoads + c) * 64 * 8 + lane * 8) = u32x4{0u, 0u, 0u, 0u};
    }
    // LDS writes done, then the barrier: the stage is complete for every
    // wave, and every wave has finished reading the stage loaded next
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    if (issued < nsteps) issue(issued++);
    const uint16_t *As = base, *Bs = base + BM * BK;
    const int kc = lane >> 4;
    bf16x8 a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      a[u] = *reinterpret_cast<const bf16x8 *>(As + ring_slot(wm + 16 * u + (lane & 15), kc) * 8);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      b[u] = *reinterpret_cast<const bf16x8 *>(Bs + ring_slot(wn + 16 * u + (lane & 15), kc) * 8);
#pragma unroll
    for (int ii = 0; ii < 4; ++ii)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
        acc[ii][jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ii], b[jj], acc[ii][jj], 0, 0, 0);
  }
  __syncthreads();   // all loads landed and all operand reads done: the ring is free
  ring_epilogue<EPI>(g, acc, S, m0, n0, z);
}

// ---- both operands K-major (opA = A[k][m], opB = B[k][n]) ----------------
// The weight gradients: sums over the rows of a batch of products of two
// row-major matrices.  Tiles, ring and epilogue are gemm_nt_kernel's; a stage
// holds 32 rows of k, 512 bytes of A and 256 of B each, and the operands, 8
// consecutive k of one column, come from two transposing LDS reads
// (ds_read_b64_tr_b16: of 16 lanes, lane 4 i + j reads columns 4 j..+4 of row i,
// and lane m receives column m of the four rows).  Chunk c of row r sits in
// place c ^ 2 (r & 3) of its row, so that the four rows of a read fall on
// distinct banks.  No operand is transposed in memory first, which took 31 to
// 35 us for each of four 57,344-row matrices; the products take as long as on
// transposed ones (65 us for 512 x 512 and 512 x 784 over 57,344 rows, the
// mean) and add the same terms in the same order.  Needs 16-byte aligned operands with
// lda, ldb, M and N multiples of 8 (N: or rows of B that hold whole chunks up to
// it), and lda and ldb below 2^26 (a stage within 4 GB).
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// byte offset in its tile (of `pitch` columns) of what the lane reads for the operand of columns col0..+16
__device__ __forceinline__ uint32_t tr_offset(int pitch, int col0, int lane) {
  const int q = lane & 3, i = (lane >> 2) & 3, row = 8 * (lane >> 4) + i;   // rows row and row + 4: the same i
  return 2u * (uint32_t)(row * pitch + ((((col0 >> 3) + (q >> 1)) ^ (i << 1)) << 3) + 4 * (q & 1));
}

// four operands' halves, in LDS behind the loads of later stages: as the
// compiler would wait for all of those before an LDS read, the reads are
// written out, with their own wait
template <int PITCH>
__device__ __forceinline__ void tr_operands(const uint32_t (&at)[4], bf16x8 (&v)[4]) {
  u32x2 lo[4], hi[4];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8\n\t"
      "ds_read_b64_tr_b16 %1, %8 offset:%12\n\t"
      "ds_read_b64_tr_b16 %2, %9\n\t"
      "ds_read_b64_tr_b16 %3, %9 offset:%12\n\t"
      "ds_read_b64_tr_b16 %4, %10\n\t"
      "ds_read_b64_tr_b16 %5, %10 offset:%12\n\t"
      "ds_read_b64_tr_b16 %6, %11\n\t"
      "ds_read_b64_tr_b16 %7, %11 offset:%12\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(lo[0]), "=&v"(hi[0]), "=&v"(lo[1]), "=&v"(hi[1]), "=&v"(lo[2]), "=&v"(hi[2]), "=&v"(lo[3]), "=&v"(hi[3])
      : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "n"(8 * PITCH)
      : "memory");
#pragma unroll
  for (int u = 0; u < 4; ++u)
    v[u] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo[u], hi[u], 0, 1, 2, 3));
}

template <int EPI>
__global__ void __launch_bounds__(kNtThreads, 4) gemm_tn_kernel(GemmArgs g, int64_t tiles_m, int64_t tiles_n) {
  __shared__ __attribute__((aligned(16))) uint16_t S[kRing * kStage];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t nb = (int64_t)gridDim.x, lin = blockIdx.x;
  const int64_t q = nb / kXcds, rem = nb % kXcds, x = lin % kXcds, i = lin / kXcds;
  const int64_t tile = x < rem ? x * (q + 1) + i : rem * (q + 1) + (x - rem) * q + i;
  const int64_t per_z = tiles_m * tiles_n, z = tile / per_z, t = tile % per_z;
  const bool m_outer = tiles_m >= tiles_n;
  const int64_t m0 = (m_outer ? t / tiles_n : t % tiles_m) * BM;
  const int64_t n0 = (m_outer ? t % tiles_n : t / tiles_m) * BN;
  const int64_t kbeg = z * g.kchunk;
  const int64_t kend = kbeg + g.kchunk < g.K ? kbeg + g.kchunk : g.K;
  const int nsteps = (int)((kend - kbeg + BK - 1) / BK);
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;

  // this thread's chunks of every stage: row of k, and bytes from the stage's
  // first row of the operand
  int row_of[kStageLoads];
  uint32_t off[kStageLoads];
#pragma unroll
  for (int c = 0; c < kStageLoads; ++c) {
    const int slot = (wave * kStageLoads + c) * 64 + lane;
    const bool isA = slot < BK * BM / 8;
    const int rs = isA ? slot : slot - BK * BM / 8, per = isA ? BM / 8 : BN / 8;
    const int r = rs / per, ch = (rs % per) ^ ((r & 3) << 1);
    const int64_t col = (isA ? m0 : n0) + 8 * ch;
    row_of[c] = r;
    // a chunk past the last column reads the first one: its outputs are not stored
    off[c] = (uint32_t)((r * (isA ? g.lda : g.ldb) + (col < (isA ? g.M : g.N) ? col : 0)) * 2);
  }
  auto issue = [&](int st) {
    uint16_t *base = S + (st % kRing) * kStage;
    const int64_t k0 = kbeg + (int64_t)st * BK;
    const int left = kend - k0 < BK ? (int)(kend - k0) : BK;   // rows past the end read row k0 and are zeroed later
#pragma unroll
    for (int c = 0; c < kStageLoads; ++c) {
      const bool isA = __builtin_amdgcn_readfirstlane((wave * kStageLoads + c) * 64) < BK * BM / 8;
      const unsigned char *from = reinterpret_cast<const unsigned char *>(isA ? g.A + k0 * g.lda : g.B + k0 * g.ldb);
      __builtin_amdgcn_global_load_lds((const void *)(from + (row_of[c] < left ? off[c] : 0u)),
                                       (lds_void *)(base + (wave * kStageLoads + c) * 64 * 8), 16, 0, 0);
    }
  };

  uint32_t at_a[4], at_b[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    at_a[u] = tr_offset(BM, wm + 16 * u, lane);
    at_b[u] = tr_offset(BN, wn + 16 * u, lane);
  }
  floatx4 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};

  int issued = 0;
  for (; issued < kRing - 1 && issued < nsteps; ++issued) issue(issued);
  for (int st = 0; st < nsteps; ++st) {
    if (issued - st - 1 >= 1) asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    uint16_t *base = S + (st % kRing) * kStage;
    if (kbeg + (int64_t)(st + 1) * BK > kend) {   // K tail: zero this thread's rows past the end
#pragma unroll
      for (int c = 0; c < kStageLoads; ++c)
        if (kbeg + (int64_t)st * BK + row_of[c] >= kend)
          *reinterpret_cast<u32x4 *>(base + (wave * kStageLoads + c) * 64 * 8 + lane * 8) = u32x4{0u, 0u, 0u, 0u};
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    if (issued < nsteps) issue(issued++);
    uint32_t stage = (uint32_t)(uintptr_t)(lds_void *)base;
    asm volatile("" : "+s"(stage));   // added here each step: the sums of all stages overflow the registers
    uint32_t pa[4], pb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      pa[u] = stage + at_a[u];
      pb[u] = stage + BK * BM * 2 + at_b[u];
    }
    bf16x8 a[4], b[4];
    tr_operands<BM>(pa, a);
    tr_operands<BN>(pb, b);
#pragma unroll
    for (int ii = 0; ii < 4; ++ii)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
        acc[ii][jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ii], b[jj], acc[ii][jj], 0, 0, 0);
  }
  __syncthreads();   // all loads landed and all operand reads done: the ring is free
  ring_epilogue<EPI>(g, acc, S, m0, n0, z);
}

// sum of `splits` FP32 slabs [M][ldc] in slab order -> out (FP32, ld = ldo)
__global__ void splitk_reduce_kernel(const float *__restrict__ part, int splits, int64_t M, int64_t N,
                                     int64_t ldp, float *__restrict__ out, int64_t ldo) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= M * N) return;
  const int64_t m = e / N, n = e % N;
  const float *p = part + m * ldp + n;
  const int64_t slab = M * ldp;
  float s = 0.f;
  int z = 0;
  for (; z + 8 <= splits; z += 8) {   // eight slabs in flight, added in order
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = p[(z + u) * slab];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += x[u];
  }
  for (; z < splits; ++z) s += p[z * slab];
  out[m * ldo + n] = s;
}

template <bool TA, bool TB>
hipError_t launch_gemm_t(const GemmArgs &g, int epi, dim3 grid, hipStream_t s) {
  switch (epi) {
    case GEMM_EPI_F32: gemm_kernel<TA, TB, GEMM_EPI_F32><<<grid, kGemmThreads, 0, s>>>(g); break;
    case GEMM_EPI_BIAS_RELU_BF16:
      gemm_kernel<TA, TB, GEMM_EPI_BIAS_RELU_BF16><<<grid, kGemmThreads, 0, s>>>(g);
      break;
    default: gemm_kernel<TA, TB, GEMM_EPI_RELU_MASK_BF16><<<grid, kGemmThreads, 0, s>>>(g); break;
  }
  return hipGetLastError();
}

// ---- small kernels around the GEMMs -------------------------------------

// out[c][r] = in[r][c] for a BF16 [R][C] matrix, rows of out padded to ldo
// (>= R) with zeros; 64 x 64 tiles through LDS (coalesced reads and writes)
__global__ void __launch_bounds__(256) transpose_bf16_kernel(const uint16_t *__restrict__ in, int64_t R, int64_t C,
                                                            uint16_t *__restrict__ out, int64_t ldo) {
  __shared__ uint16_t t[64][65];
  const int64_t r0 = (int64_t)blockIdx.x * 64, c0 = (int64_t)blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int i = ty; i < 64; i += 4) {
    const int64_t r = r0 + i, c = c0 + tx;
    t[i][tx] = (r < R && c < C) ? in[r * C + c] : (uint16_t)0;
  }
  __syncthreads();
  for (int i = ty; i < 64; i += 4) {
    const int64_t c = c0 + i, r = r0 + tx;
    if (c < C && r < ldo) out[c * ldo + r] = t[tx][i];
  }
}

__global__ void f32_to_bf16_kernel(const float *__restrict__ x, int64_t n, uint16_t *__restrict__ y) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) y[e] = f2bf(x[e]);
}

// out[r][0..ldo) = X[rows[r]][0..N) and zeros (rows NULL: X[r]), by 16-byte
// chunks of out; X's rows start at any element
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));

__global__ void gather_rows_kernel(const uint16_t *__restrict__ X, int64_t N, const int32_t *__restrict__ rows,
                                   int64_t R, uint16_t *__restrict__ out, int64_t ldo) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t cpr = ldo / 8;   // chunks per row
  if (e >= R * cpr) return;
  const int64_t r = e / cpr, k = (e - r * cpr) * 8;
  const uint16_t *x = X + (rows ? (int64_t)rows[r] : r) * N + k;
  u32x4 v = u32x4{0u, 0u, 0u, 0u};
  if (k + 8 <= N)
    v = *reinterpret_cast<const u32x4u *>(x);
  else
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (k + j < N) v[j >> 1] |= (uint32_t)x[j] << (16 * (j & 1));
  *reinterpret_cast<u32x4 *>(out + r * ldo + k) = v;
}

// Z[r][o] = b3[o] + sum_k H[r][k] W3[o][k], o < 2 (one wavefront per row;
// with vec, K % 8 == 0 and 16-byte aligned H and W3, each lane takes 8
// consecutive k per 16-byte load)
__global__ void __launch_bounds__(256) head_forward_kernel(const uint16_t *__restrict__ H, int64_t R, int K,
                                                           const uint16_t *__restrict__ W3,
                                                           const float *__restrict__ b3, float *__restrict__ Z,
                                                           bool vec) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= R) return;
  float s0 = 0.f, s1 = 0.f;
  if (vec) {
    for (int k = 8 * lane; k < K; k += 512) {
      const U16x8 h = *reinterpret_cast<const U16x8 *>(H + r * K + k);
      const U16x8 w0 = *reinterpret_cast<const U16x8 *>(W3 + k);
      const U16x8 w1 = *reinterpret_cast<const U16x8 *>(W3 + K + k);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        s0 += bf2f(h.v[j]) * bf2f(w0.v[j]);
        s1 += bf2f(h.v[j]) * bf2f(w1.v[j]);
      }
    }
  } else {
    for (int k = lane; k < K; k += 64) {
      const float h = bf2f(H[r * K + k]);
      s0 += h * bf2f(W3[k]);
      s1 += h * bf2f(W3[K + k]);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    s0 += __shfl_xor(s0, o, 64);
    s1 += __shfl_xor(s1, o, 64);
  }
  if (lane == 0) {
    Z[2 * r] = s0 + b3[0];
    Z[2 * r + 1] = s1 + b3[1];
  }
}

// Column sums of a BF16 matrix X [R][J], J even (the bias gradients), as the
// sums of kBiasLanes lanes: lane t takes rows 8 t..8 t + 7 of every 8 kBiasLanes,
// in order, and a tree adds the lanes.  bias_lanes_kernel: a wavefront per lane
// and 128 columns, 32 rows in flight: part[t][J].
constexpr int kBiasLanes = 256;
constexpr int kBiasAhead = 4;   // groups of 8 rows in flight (the loads one by one: 70 us for 57,344 x 512, so 12)

__global__ void __launch_bounds__(256) bias_lanes_kernel(const uint16_t *__restrict__ X, int64_t R, int64_t J,
                                                        float *__restrict__ part) {
  const int t = (int)blockIdx.y * 4 + (threadIdx.x >> 6);
  const int64_t j = ((int64_t)blockIdx.x * 64 + (threadIdx.x & 63)) * 2;
  if (j >= J) return;
  float s0 = 0.f, s1 = 0.f;
  int64_t r0 = 8 * t;
  for (; r0 + 8 * kBiasLanes * (kBiasAhead - 1) + 8 <= R; r0 += 8 * kBiasLanes * kBiasAhead) {
    const uint16_t *p = X + r0 * J + j;
    uint32_t x[kBiasAhead * 8];
#pragma unroll
    for (int g = 0; g < kBiasAhead; ++g)
#pragma unroll
      for (int u = 0; u < 8; ++u) x[g * 8 + u] = *reinterpret_cast<const uint32_t *>(p + (g * 8 * kBiasLanes + u) * J);
    __builtin_amdgcn_sched_barrier(0);   // all on their way before the first is added
#pragma unroll
    for (int u = 0; u < kBiasAhead * 8; ++u) {
      s0 += __uint_as_float(x[u] << 16);
      s1 += __uint_as_float(x[u] & 0xffff0000u);
    }
  }
  for (; r0 < R; r0 += 8 * kBiasLanes)
    for (int u = 0; u < 8 && r0 + u < R; ++u) {
      const uint32_t x = *reinterpret_cast<const uint32_t *>(X + (r0 + u) * J + j);
      s0 += __uint_as_float(x << 16);
      s1 += __uint_as_float(x & 0xffff0000u);
    }
  part[t * J + j] = s0;
  part[t * J + j + 1] = s1;
}

// out[j] = the tree sum of part[0..kBiasLanes)[j]: lane t adds lane t + w, w = 128, 64, ...
__global__ void __launch_bounds__(kBiasLanes) bias_tree_kernel(const float *__restrict__ part, int64_t J,
                                                              float *__restrict__ out) {
  __shared__ float red[kBiasLanes][8];
  const int t = threadIdx.x;
  const int64_t j0 = (int64_t)blockIdx.x * 8;
#pragma unroll
  for (int e = 0; e < 8; ++e) red[t][e] = j0 + e < J ? part[t * J + j0 + e] : 0.f;
  __syncthreads();
  for (int w = kBiasLanes / 2; w > 0; w >>= 1) {
    if (t < w)
#pragma unroll
      for (int e = 0; e < 8; ++e) red[t][e] += red[t + w][e];
    __syncthreads();
  }
  if (t < 8 && j0 + t < J) out[j0 + t] = red[0][t];
}

// Backward of the head on kColsumRows rows and 128 columns: the input gradient
//   dH[r][k] = (dZ[r][0] W3[0][k] + dZ[r][1] W3[1][k]) * [H[r][k] > 0]  -> BF16
// and, while H is at hand, the chunk's column sums of dZ[.][0] x H and
// dZ[.][1] x H (dW3) into part[chunk][2 K].  The sums' order is colsum_kernel's.
// Needs K % 4 == 0 and 8-byte aligned H and dH.  Bound by memory: H read and dH
// written once, 57,344 x 512 in 30 us, where two passes over H took 48.
__global__ void __launch_bounds__(kColsumThreads) head_backward_kernel(const float *__restrict__ dZ,
                                                           const uint16_t *__restrict__ W3,
                                                           const uint16_t *__restrict__ H, int64_t R, int K,
                                                           uint16_t *__restrict__ dH, float *__restrict__ part) {
  constexpr int V = 4;
  __shared__ float red[kColsumLanes][32 * V + 1];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int k0 = (int)(blockIdx.x * 32 + tx) * V;
  const int64_t r0 = (int64_t)blockIdx.y * kColsumRows;
  const int64_t r1 = r0 + kColsumRows < R ? r0 + kColsumRows : R;
  float sum[2][V], w0[V], w1[V];
#pragma unroll
  for (int e = 0; e < V; ++e) {
    sum[0][e] = sum[1][e] = 0.f;
    w0[e] = k0 < K ? bf2f(W3[k0 + e]) : 0.f;
    w1[e] = k0 < K ? bf2f(W3[K + k0 + e]) : 0.f;
  }
  auto load = [&](int64_t r) { return *reinterpret_cast<const U16x4 *>(H + r * K + k0); };
  auto take = [&](int64_t r, U16x4 h, float g0, float g1) {
#pragma unroll
    for (int e = 0; e < V; ++e) {
#pragma clang fp contract(off)
      // the roundings are written out: the compiler's own fusions vary with the code around them
      const float x = bf2f(h.v[e]);
      const float g = fmaf(g0, w0[e], g1 * w1[e]);
      h.v[e] = f2bf(x > 0.f ? g : 0.f);
      sum[0][e] = sum[0][e] + g0 * x;
      sum[1][e] = sum[1][e] + g1 * x;
    }
    *reinterpret_cast<U16x4 *>(dH + r * K + k0) = h;
  };
  if (k0 < K) {
    constexpr int kAhead = 8;
    int64_t r = r0 + ty;
    for (; r + (kAhead - 1) * kColsumLanes < r1; r += kAhead * kColsumLanes) {
      U16x4 h[kAhead];
      float g0[kAhead], g1[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        h[u] = load(r + u * kColsumLanes);
        g0[u] = dZ[2 * (r + u * kColsumLanes)];
        g1[u] = dZ[2 * (r + u * kColsumLanes) + 1];
      }
      __builtin_amdgcn_sched_barrier(0);   // all on their way before the first is used
#pragma unroll
      for (int u = 0; u < kAhead; ++u) take(r + u * kColsumLanes, h[u], g0[u], g1[u]);
    }
    for (; r < r1; r += kColsumLanes) take(r, load(r), dZ[2 * r], dZ[2 * r + 1]);
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    __syncthreads();
#pragma unroll
    for (int e = 0; e < V; ++e) red[ty][tx * V + e] = sum[q][e];
    __syncthreads();
    for (int c = threadIdx.x; c < 32 * V; c += kColsumThreads) {
      const int k = (int)blockIdx.x * 32 * V + c;
      if (k >= K) continue;
      float t = red[0][c];
#pragma unroll
      for (int y = 1; y < kColsumLanes; ++y) t += red[y][c];
      part[(int64_t)blockIdx.y * 2 * K + (int64_t)q * K + k] = t;
    }
  }
}

// column sums of the FP32 matrix X [R][J] over row chunks (the head's bias
// gradient, and the later levels of a sum): part[c][j] = sum_{r in chunk c} X[r][j]
// A block of kColsumLanes x 32 threads covers 32 V-column groups of one chunk
// of kColsumRows rows: row lane ty sums rows ty, ty + kColsumLanes, ... in
// order, then the lane sums are added in order of ty (deterministic).  V = 4
// needs J a multiple of 4 and a 16-byte aligned source; eight rows in flight.
template <int V>
__global__ void __launch_bounds__(kColsumThreads) colsum_kernel(const float *__restrict__ X, int64_t R, int64_t J,
                                                                float *__restrict__ part) {
  __shared__ float red[kColsumLanes][32 * V + 1];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int64_t j0 = ((int64_t)blockIdx.x * 32 + tx) * V;
  const int64_t r0 = (int64_t)blockIdx.y * kColsumRows;
  const int64_t r1 = r0 + kColsumRows < R ? r0 + kColsumRows : R;
  float acc[V];
#pragma unroll
  for (int e = 0; e < V; ++e) acc[e] = 0.f;
  if (j0 < J) {
#pragma unroll 8
    for (int64_t r = r0 + ty; r < r1; r += kColsumLanes) {
      const float *x = X + r * J + j0;
      if (V == 4) {
        const floatx4 v = *reinterpret_cast<const floatx4 *>(x);
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] += v[e];
      } else {
        acc[0] += x[0];
      }
    }
  }
#pragma unroll
  for (int e = 0; e < V; ++e) red[ty][tx * V + e] = acc[e];
  __syncthreads();
  if (ty == 0 && j0 < J) {
#pragma unroll
    for (int e = 0; e < V; ++e) {
      float t = red[0][tx * V + e];
#pragma unroll
      for (int q = 1; q < kColsumLanes; ++q) t += red[q][tx * V + e];
      part[(int64_t)blockIdx.y * J + j0 + e] = t;
    }
  }
}

// Adam with bias correction 1/(1 - beta^t); refreshes the BF16 copy
__global__ void adam_kernel(float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m,
                            float *__restrict__ v, uint16_t *__restrict__ w16, int64_t n, float lr, float b1,
                            float b2, float eps, float c1, float c2, float gscale) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const float gr = g[e] * gscale;
  const float mm = b1 * m[e] + (1.f - b1) * gr;
  const float vv = b2 * v[e] + (1.f - b2) * gr * gr;
  m[e] = mm;
  v[e] = vv;
  const float wn = w[e] - lr * (mm / c1) / (sqrtf(vv / c2) + eps);
  w[e] = wn;
  w16[e] = f2bf(wn);
}

// Glorot-uniform weights U(-s, s), s = sqrt(6 / (fan_in + fan_out)), from a
// SplitMix64 counter stream; biases zero
__global__ void glorot_kernel(float *__restrict__ w, int64_t n, int fan_in, int fan_out, uint64_t seed,
                              uint64_t offset) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  uint64_t z = seed ^ (offset + (uint64_t)e) * 0x9e3779b97f4a7c15ull;
  z += 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  z ^= z >> 31;
  const float u = (float)(z >> 40) * (1.0f / 16777216.0f);   // [0, 1)
  const float s = sqrtf(6.0f / (float)(fan_in + fan_out));
  w[e] = (2.f * u - 1.f) * s;
}

}  // namespace

hipError_t launch_gemm_bf16(const GemmArgs &g0, int ta, int tb, int epi, int splits, hipStream_t s) {
  GemmArgs g = g0;
  if (splits < 1) splits = 1;
  g.kchunk = ((g.K + splits - 1) / splits + NTK - 1) / NTK * NTK;
  if (g.kchunk < NTK) g.kchunk = NTK;
  splits = (int)((g.K + g.kchunk - 1) / g.kchunk);
  if (splits < 1) splits = 1;
  const bool nt = !ta && tb && g.vec_a && g.vec_b && g.K % 8 == 0;
  const bool tn_ok = ta && !tb && g.vec_a && g.vec_b && g.M % 8 == 0 && (g.N % 8 == 0 || g.whole_b) &&
                     g.lda < (int64_t)1 << 26 && g.ldb < (int64_t)1 << 26;
  if (nt || tn_ok) {
    const int64_t tm = (g.M + BM - 1) / BM, tn = (g.N + BN - 1) / BN, nb = tm * tn * splits;
    if (nb > INT32_MAX) return hipErrorInvalidValue;
    if (tn_ok) {
      switch (epi) {
        case GEMM_EPI_F32: gemm_tn_kernel<GEMM_EPI_F32><<<(unsigned)nb, kNtThreads, 0, s>>>(g, tm, tn); break;
        case GEMM_EPI_BIAS_RELU_BF16:
          gemm_tn_kernel<GEMM_EPI_BIAS_RELU_BF16><<<(unsigned)nb, kNtThreads, 0, s>>>(g, tm, tn);
          break;
        default: gemm_tn_kernel<GEMM_EPI_RELU_MASK_BF16><<<(unsigned)nb, kNtThreads, 0, s>>>(g, tm, tn); break;
      }
      return hipGetLastError();
    }
    switch (epi) {
      case GEMM_EPI_F32: gemm_nt_kernel<GEMM_EPI_F32><<<(unsigned)nb, kNtThreads, 0, s>>>(g, tm, tn); break;
      case GEMM_EPI_BIAS_RELU_BF16:
        gemm_nt_kernel<GEMM_EPI_BIAS_RELU_BF16><<<(unsigned)nb, kNtThreads, 0, s>>>(g, tm, tn);
        break;
      default: gemm_nt_kernel<GEMM_EPI_RELU_MASK_BF16><<<(unsigned)nb, kNtThreads, 0, s>>>(g, tm, tn); break;
    }
    return hipGetLastError();
  }
  dim3 grid((unsigned)((g.N + TN - 1) / TN), (unsigned)((g.M + TM - 1) / TM), (unsigned)splits);
  if (!ta && !tb) return launch_gemm_t<false, false>(g, epi, grid, s);
  if (!ta && tb) return launch_gemm_t<false, true>(g, epi, grid, s);
  if (ta && !tb) return launch_gemm_t<true, false>(g, epi, grid, s);
  return launch_gemm_t<true, true>(g, epi, grid, s);
}

int gemm_splits_used(int64_t K, int splits) {
  if (splits < 1) splits = 1;
  int64_t kchunk = ((K + splits - 1) / splits + NTK - 1) / NTK * NTK;
  if (kchunk < NTK) kchunk = NTK;
  const int64_t used = (K + kchunk - 1) / kchunk;
  return (int)(used < 1 ? 1 : used);
}

hipError_t launch_splitk_reduce(const float *part, int splits, int64_t M, int64_t N, int64_t ldp, float *out,
                                int64_t ldo, hipStream_t s) {
  splitk_reduce_kernel<<<grid_for(M * N), kBlock, 0, s>>>(part, splits, M, N, ldp, out, ldo);
  return hipGetLastError();
}

hipError_t launch_transpose_bf16(const uint16_t *in, int64_t R, int64_t C, uint16_t *out, int64_t ldo,
                                 hipStream_t s) {
  if (ldo == 0 || C == 0) return hipSuccess;
  if (ldo < R || (C + 63) / 64 > 65535 || (ldo + 63) / 64 > INT32_MAX) return hipErrorInvalidValue;
  transpose_bf16_kernel<<<dim3((unsigned)((ldo + 63) / 64), (unsigned)((C + 63) / 64)), 256, 0, s>>>(in, R, C, out,
                                                                                                    ldo);
  return hipGetLastError();
}

hipError_t launch_f32_to_bf16(const float *x, int64_t n, uint16_t *y, hipStream_t s) {
  f32_to_bf16_kernel<<<grid_for(n), kBlock, 0, s>>>(x, n, y);
  return hipGetLastError();
}

hipError_t launch_gather_rows(const uint16_t *X, int64_t N, const int32_t *rows, int64_t R, uint16_t *out,
                              int64_t ldo, hipStream_t s) {
  if (ldo % 8 || (reinterpret_cast<uintptr_t>(out) & 15)) return hipErrorInvalidValue;
  gather_rows_kernel<<<grid_for(R * (ldo / 8)), kBlock, 0, s>>>(X, N, rows, R, out, ldo);
  return hipGetLastError();
}

hipError_t launch_head_forward(const uint16_t *H, int64_t R, int K, const uint16_t *W3, const float *b3, float *Z,
                               hipStream_t s) {
  const bool vec = K % 8 == 0 && (reinterpret_cast<uintptr_t>(H) & 15) == 0 &&
                   (reinterpret_cast<uintptr_t>(W3) & 15) == 0;
  head_forward_kernel<<<grid_for(R, 4), 256, 0, s>>>(H, R, K, W3, b3, Z, vec);
  return hipGetLastError();
}

int64_t colsum_workspace(int64_t R, int64_t J) {
  const int64_t c0 = (R + kColsumRows - 1) / kColsumRows;
  return (c0 + (c0 + kColsumRows - 1) / kColsumRows) * J;
}

// Column sums as a tree: each level sums kColsumRows consecutive rows into
// partials [ceil(rows / kColsumRows)][J], until one row is left (written to
// out).  Levels ping-pong between two regions of ws.
hipError_t launch_colsum(const float *X, int64_t R, int64_t J, float *ws, float *out, hipStream_t s) {
  if (R < 1 || (R + kColsumRows - 1) / kColsumRows > 65535) return hipErrorInvalidValue;
  const int64_t c0 = (R + kColsumRows - 1) / kColsumRows;
  float *buf[2] = {ws, ws + c0 * J};
  const float *src = X;
  int64_t rows = R;
  for (int level = 0;; ++level) {
    const int64_t chunks = (rows + kColsumRows - 1) / kColsumRows;
    float *dst = chunks == 1 ? out : buf[level & 1];
    const bool vec4 = J % 4 == 0 && (reinterpret_cast<uintptr_t>(src) & 15) == 0;
    if (vec4)
      colsum_kernel<4><<<dim3((unsigned)((J / 4 + 31) / 32), (unsigned)chunks), kColsumThreads, 0, s>>>(src, rows, J, dst);
    else
      colsum_kernel<1><<<dim3((unsigned)((J + 31) / 32), (unsigned)chunks), kColsumThreads, 0, s>>>(src, rows, J, dst);
    if (chunks == 1) break;
    src = dst;
    rows = chunks;
  }
  return hipGetLastError();
}

int64_t bias_workspace(int64_t J) { return kBiasLanes * J; }

hipError_t launch_bias_sum(const uint16_t *X, int64_t R, int64_t J, float *ws, float *out, hipStream_t s) {
  if (R < 1 || J < 2 || J % 2 || (reinterpret_cast<uintptr_t>(X) & 3)) return hipErrorInvalidValue;
  bias_lanes_kernel<<<dim3((unsigned)((J + 127) / 128), kBiasLanes / 4), 256, 0, s>>>(X, R, J, ws);
  bias_tree_kernel<<<(unsigned)((J + 7) / 8), kBiasLanes, 0, s>>>(ws, J, out);
  return hipGetLastError();
}

hipError_t launch_head_backward(const float *dZ, const uint16_t *W3, const uint16_t *H, int64_t R, int K,
                                uint16_t *dH, float *ws, float *out, hipStream_t s) {
  if (R < 1 || (R + kColsumRows - 1) / kColsumRows > 65535) return hipErrorInvalidValue;
  const int64_t chunks = (R + kColsumRows - 1) / kColsumRows, J = 2 * (int64_t)K;
  float *part = chunks == 1 ? out : ws;
  if (K % 4 || ((reinterpret_cast<uintptr_t>(H) | reinterpret_cast<uintptr_t>(dH)) & 7)) return hipErrorInvalidValue;
  head_backward_kernel<<<dim3((unsigned)((K / 4 + 31) / 32), (unsigned)chunks), kColsumThreads, 0, s>>>(dZ, W3, H, R, K,
                                                                                                      dH, part);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || chunks == 1) return e;
  return launch_colsum(part, chunks, J, ws + chunks * J, out, s);
}

hipError_t launch_adam(float *w, const float *g, float *m, float *v, uint16_t *w16, int64_t n, float lr, float b1,
                       float b2, float eps, int64_t t, float gscale, hipStream_t s) {
  const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
  adam_kernel<<<grid_for(n), kBlock, 0, s>>>(w, g, m, v, w16, n, lr, b1, b2, eps, c1, c2, gscale);
  return hipGetLastError();
}

hipError_t launch_glorot(float *w, int64_t n, int fan_in, int fan_out, uint64_t seed, uint64_t offset,
                         hipStream_t s) {
  glorot_kernel<<<grid_for(n), kBlock, 0, s>>>(w, n, fan_in, fan_out, seed, offset);
  return hipGetLastError();
}

}  // namespace ivhd

namespace ivhd {
namespace {

// rows of one training batch: B sources s_b = (a (off + b) + c0) mod M, then
// their nn targets (an absent slot repeats the source, which adds nothing to
// the stress or its gradient), then their rn targets
__global__ void batch_rows_kernel(const int32_t *__restrict__ nn_idx, int nn, const int32_t *__restrict__ rn_idx,
                                  int rn, int64_t M, int64_t B, uint64_t a, uint64_t c0, int64_t off,
                                  int32_t *__restrict__ rows) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const int64_t src = (int64_t)((a * (uint64_t)(off + b) + c0) % (uint64_t)M);
  rows[b] = (int32_t)src;
  for (int q = 0; q < nn; ++q) {
    const int32_t j = nn_idx[src * nn + q];
    rows[B + b * nn + q] = j >= 0 ? j : (int32_t)src;
  }
  for (int q = 0; q < rn; ++q) rows[B + B * nn + b * rn + q] = rn_idx[src * rn + q];
}

// the fixed local edge lists of a batch: source b's nn edges point at rows
// B + b*nn + q, its rn edges at rows B + B*nn + b*rn + q; other rows have none
__global__ void batch_plan_kernel(int64_t B, int nn, int rn, int32_t *__restrict__ lnn, int32_t *__restrict__ lrn) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t R = B * (1 + nn + rn);
  if (r >= R) return;
  for (int q = 0; q < nn; ++q) lnn[r * nn + q] = r < B ? (int32_t)(B + r * nn + q) : -1;
  for (int q = 0; q < rn; ++q) lrn[r * rn + q] = r < B ? (int32_t)(B + B * nn + r * rn + q) : -1;
}

}  // namespace

hipError_t launch_batch_rows(const int32_t *nn_idx, int nn, const int32_t *rn_idx, int rn, int64_t M, int64_t B,
                             uint64_t a, uint64_t c0, int64_t off, int32_t *rows, hipStream_t s) {
  batch_rows_kernel<<<grid_for(B), kBlock, 0, s>>>(nn_idx, nn, rn_idx, rn, M, B, a, c0, off, rows);
  return hipGetLastError();
}

hipError_t launch_batch_plan(int64_t B, int nn, int rn, int32_t *lnn, int32_t *lrn, hipStream_t s) {
  batch_plan_kernel<<<grid_for(B * (1 + nn + rn)), kBlock, 0, s>>>(B, nn, rn, lnn, lrn);
  return hipGetLastError();
}

}  // namespace ivhd
