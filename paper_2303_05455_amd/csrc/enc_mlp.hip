// The encoder's forward pass in one kernel: N-D -> h1 -> h2 -> 2 for a tile of
// rows whose hidden activations stay in LDS.
//
// Layer by layer, the pass moved each activation matrix out to memory and in
// again (57,344 rows of 512: 59 MB each way) between products that read
// 0.5 KB of operands from LDS per MFMA and were bound by that.  Here a block
// of eight wavefronts takes 16 RT rows and all columns, 64 a wavefront:
//   * a wavefront's weights are its own, so they go from L2 to registers, not
//     through LDS: packed in the order of the matrix instruction's lanes
//     (pack_kernel), a load is one contiguous KB, and two or four steps of K
//     are in flight;
//   * the rows are shared by the eight: K in stages of 128 through registers
//     into a ring of two LDS stages, one barrier each; a wavefront reads RT
//     operands from LDS for 4 RT MFMAs;
//   * the weights are the instruction's first operand, so that a lane's four
//     results are consecutive columns of one row: after bias, ReLU and
//     rounding they go to LDS as 8 bytes, in place of the ring, and are the
//     next layer's operand there: layer 2 needs no barrier in its loop;
//   * the head's two dot products read the second activations from LDS, a
//     wavefront per row.
// Each output adds the same products in the same order as gemm_nt_kernel's and
// head_forward_kernel's (v_mfma_f32_16x16x32_bf16 over steps of 32), and the
// results are the same bit for bit.
//
// Bound: the matrix units, at the clock they leave (1.7 GHz in dense loops):
// 200,000 rows of 784 -> 512 -> 512 -> 2 took 549 us as two products and the
// head for each 57,344 rows, and take 309 (865 TFLOP/s); storing the
// activations too, 57,344 rows take 113 us against 153.  Two steps of weights
// in flight and seven row tiles fit the 256 registers of two wavefronts a SIMD:
// four steps spill (477 us), six row tiles lose a sixth of the reuse (394 us).
#include "enc_internal.h"

namespace ivhd {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));   // 16 bytes at any element

constexpr int kWide = 512;            // columns of a block: eight wavefronts of 64
constexpr int kMlpThreads = 512;
constexpr int kStageK = 128;          // K of an LDS stage: four steps of 32
constexpr int kSteps = kStageK / 32;

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// to nearest even, a NaN quietened: the conversion instruction's results, which
// the eight integer operations of doing it by hand have for every float
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// P[tile][step][lane][8] = W[16 tile + lane % 16][32 step + 8 (lane / 16) + 0..7],
// zero outside W [n][k]; kWide / 16 tiles
struct PackArgs {
  const uint16_t *W;
  uint16_t *P;
  int n, k, steps;
};
__global__ void pack_kernel(PackArgs first, PackArgs second) {   // blockIdx.y: which
  const PackArgs &a = blockIdx.y ? second : first;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)(kWide / 16) * a.steps * 64) return;
  const int lane = (int)(t & 63), step = (int)((t >> 6) % a.steps), tile = (int)((t >> 6) / a.steps);
  const int row = 16 * tile + (lane & 15), k0 = 32 * step + 8 * (lane >> 4);
  u32x4 v = u32x4{0u, 0u, 0u, 0u};
  if (row < a.n) {
    const uint16_t *w = a.W + (int64_t)row * a.k + k0;
    if (k0 + 8 <= a.k)
      v = *reinterpret_cast<const u32x4u *>(w);
    else
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (k0 + e < a.k) v[e >> 1] |= (uint32_t)w[e] << (16 * (e & 1));
  }
  *reinterpret_cast<u32x4 *>(a.P + t * 8) = v;
}

// 16-byte chunk c of row m of an LDS matrix of `pitch` chunks a row: the rows
// that eight lanes read at a time fall on distinct banks
__device__ __forceinline__ int chunk_at(int m, int c, int pitch) { return (m * pitch + (c ^ (m & 7))) * 8; }

template <int RT>
struct Mlp {
  static constexpr int kRows = 16 * RT;
  static constexpr int kRing = kRows * kStageK;              // halves of a stage
  static constexpr int kFetch = (RT + 1) / 2;                // 16-byte chunks per thread and stage
  static constexpr int kAhead = RT > 6 ? 2 : 4;              // steps of weights in flight: what the registers hold
  static constexpr int kLds = kRows * kWide > 2 * kRing ? kRows * kWide : 2 * kRing;
};

template <int RT, bool STORE>
__global__ void __launch_bounds__(kMlpThreads, 2) mlp_forward_kernel(MlpArgs a) {
  using T = Mlp<RT>;
  __shared__ __attribute__((aligned(16))) uint16_t S[T::kLds];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * T::kRows;
  const int lr = lane & 15, lk = lane >> 4;   // row and chunk of K of the lane's operands
  const int steps1 = (a.n_in + 31) / 32, steps2 = (a.h1 + 31) / 32;
  const int stages1 = (steps1 + kSteps - 1) / kSteps;

  bf16x8 w[T::kAhead][4];
  auto load_w = [&](int u, const uint16_t *P, int steps, int step) {
    step = step < steps ? step : steps - 1;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      w[u % T::kAhead][j] = *reinterpret_cast<const bf16x8 *>(P + ((int64_t)(4 * wave + j) * steps + step) * 512 + lane * 8);
  };

  u32x4 x[T::kFetch];
  const unsigned char *Xb = reinterpret_cast<const unsigned char *>(a.X + r0 * a.ldx);
  const uint32_t last = (uint32_t)(a.R - 1 - r0 < T::kRows - 1 ? a.R - 1 - r0 : T::kRows - 1);
  uint32_t at[T::kFetch];   // byte of the thread's chunk of stage 0 (its rows are within 128 x 128 KB)
#pragma unroll
  for (int i = 0; i < T::kFetch; ++i) {
    const uint32_t m = (uint32_t)(tid + kMlpThreads * i) >> 4;
    at[i] = ((m < last ? m : last) * (uint32_t)a.ldx + (tid & 15) * 8u) * 2u;
  }
  auto fetch = [&](int st) {
    const int k = st * kStageK + (tid & 15) * 8;
    const bool in = k < a.n_in;
    // a row's last chunk that is not whole (only where the pitch is not a
    // multiple of 8): its elements are the last of the eight at the row's end
    const int past = k + 8 - a.ldx;
    const uint32_t step = (uint32_t)(st * kStageK - (in && past > 0 ? past : 0)) * 2u;
#pragma unroll
    for (int i = 0; i < T::kFetch; ++i) {
      x[i] = *reinterpret_cast<const u32x4u *>(Xb + (in ? at[i] + step : 0u));
      if (!in) x[i] = u32x4{0u, 0u, 0u, 0u};
    }
    if (in && past > 0) {
#pragma unroll
      for (int i = 0; i < T::kFetch; ++i) {
        uint64_t lo = (uint64_t)x[i][1] << 32 | x[i][0], hi = (uint64_t)x[i][3] << 32 | x[i][2];
        const int sh = 16 * past;   // 16 to 112
        lo = sh >= 64 ? hi >> (sh - 64) : lo >> sh | hi << (64 - sh);
        hi = sh >= 64 ? 0 : hi >> sh;
        x[i] = u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
      }
    }
  };
  auto put = [&](int st) {
    uint16_t *ring = S + (st & 1) * T::kRing;
#pragma unroll
    for (int i = 0; i < T::kFetch; ++i) {
      const int id = tid + kMlpThreads * i, m = id >> 4;
      if (RT % 2 == 0 || m < T::kRows) *reinterpret_cast<u32x4 *>(ring + chunk_at(m, id & 15, kStageK / 8)) = x[i];
    }
  };

  floatx4 acc[RT][4];
  auto clear = [&]() {
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[t][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  };
  auto multiply = [&](int u, const uint16_t *rows, int chunk, int pitch) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const bf16x8 b = *reinterpret_cast<const bf16x8 *>(rows + chunk_at(16 * t + lr, chunk, pitch));
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[u % T::kAhead][j], b, acc[t][j], 0, 0, 0);
    }
  };
  // bias, ReLU, rounding; the block's activations into S, zero past column n
  auto activate = [&](const float *bias, int n) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int col = 64 * wave + 16 * j + 4 * lk;
      const bool in = col < n;   // n is a multiple of 8: the four columns are all in or all out
      floatx4 b = floatx4{0.f, 0.f, 0.f, 0.f};
      if (in)
#pragma unroll
        for (int e = 0; e < 4; ++e) b[e] = bias[col + e];
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        uint32_t o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = in ? f2bf(fmaxf(acc[t][j][e] + b[e], 0.f)) : 0u;
        *reinterpret_cast<u32x2 *>(S + chunk_at(16 * t + lr, col >> 3, kWide / 8) + (col & 4)) =
            u32x2{o[0] | o[1] << 16, o[2] | o[3] << 16};
      }
    }
  };
  auto store = [&](uint16_t *out, int n) {
    const int cpr = n / 8;
    for (int id = tid; id < T::kRows * cpr; id += kMlpThreads) {
      const int m = id / cpr, c = id - m * cpr;
      if (r0 + m < a.R)
        *reinterpret_cast<u32x4 *>(out + (r0 + m) * n + c * 8) =
            *reinterpret_cast<const u32x4 *>(S + chunk_at(m, c, kWide / 8));
    }
  };

  clear();
  fetch(0);
#pragma unroll
  for (int u = 0; u < T::kAhead; ++u) load_w(u, a.W1p, steps1, u);
  put(0);
  if (stages1 > 1) fetch(1);
  __syncthreads();
  for (int st = 0; st < stages1; ++st) {
    const uint16_t *ring = S + (st & 1) * T::kRing;
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      const int step = st * kSteps + u;
      if (step < steps1) multiply(u, ring, 4 * u + lk, kStageK / 8);
      // the steps of layer 2 follow those of layer 1's last stage
      if (u + T::kAhead < kSteps || st + 1 < stages1) load_w(u, a.W1p, steps1, step + T::kAhead);
      else load_w(u, a.W2p, steps2, u + T::kAhead - kSteps);
      if (u == 1 && st + 1 < stages1) {   // the other stage was last read before the last barrier
        put(st + 1);
        if (st + 2 < stages1) fetch(st + 2);
      }
    }
    __syncthreads();
  }
  activate(a.b1, a.h1);
  __syncthreads();
  if (STORE) store(a.A1, a.h1);
  clear();
  for (int s0 = 0; s0 < steps2; s0 += kSteps)
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      if (s0 + u < steps2) multiply(u, S, 4 * (s0 + u) + lk, kWide / 8);
      load_w(u, a.W2p, steps2, s0 + u + T::kAhead);
    }
  __syncthreads();
  activate(a.b2, a.h2);
  __syncthreads();
  if (STORE) store(a.A2, a.h2);
  float w0[8], w1[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int k = 8 * lane + j;
    w0[j] = k < a.h2 ? bf2f(a.W3[k]) : 0.f;
    w1[j] = k < a.h2 ? bf2f(a.W3[a.h2 + k]) : 0.f;
  }
  const float b30 = a.b3[0], b31 = a.b3[1];
#pragma unroll 2
  for (int m = wave; m < T::kRows; m += kMlpThreads / 64) {
    const u32x4 h = *reinterpret_cast<const u32x4 *>(S + chunk_at(m, lane, kWide / 8));
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float hj = bf2f((uint16_t)(h[j >> 1] >> (16 * (j & 1))));
      s0 += hj * w0[j];
      s1 += hj * w1[j];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      s0 += __shfl_xor(s0, o, 64);
      s1 += __shfl_xor(s1, o, 64);
    }
    if (lane == 0 && r0 + m < a.R) {
      a.Z[2 * (r0 + m)] = s0 + b30;
      a.Z[2 * (r0 + m) + 1] = s1 + b31;
    }
  }
}

template <int RT>
hipError_t launch_rt(const MlpArgs &a, hipStream_t s) {
  const unsigned grid = (unsigned)((a.R + 16 * RT - 1) / (16 * RT));
  if (a.A1) mlp_forward_kernel<RT, true><<<grid, kMlpThreads, 0, s>>>(a);
  else mlp_forward_kernel<RT, false><<<grid, kMlpThreads, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace

bool mlp_ok(int n_in, int h1, int h2) {
  return n_in >= 8 && h1 % 8 == 0 && h2 % 8 == 0 && h1 <= kWide && h2 <= kWide && h1 > kWide - 64 && h2 > kWide - 64;
}

int64_t mlp_pack_elems(int n_in, int h1) { return ((n_in + 31) / 32 + (h1 + 31) / 32) * (int64_t)(kWide * 32); }

hipError_t launch_mlp_forward(MlpArgs a, const uint16_t *W1, const uint16_t *W2, uint16_t *pack, hipStream_t s) {
  const int steps1 = (a.n_in + 31) / 32, steps2 = (a.h1 + 31) / 32;
  uint16_t *p2 = pack + (int64_t)steps1 * kWide * 32;
  const int most = steps1 > steps2 ? steps1 : steps2;
  pack_kernel<<<dim3(grid_for((int64_t)(kWide / 16) * most * 64), 2), kBlock, 0, s>>>(
      PackArgs{W1, pack, a.h1, a.n_in, steps1}, PackArgs{W2, p2, a.h2, a.h1, steps2});
  a.W1p = pack;
  a.W2p = p2;
  // rows of a block: the fewest rounds of the 256 CUs, weighted by a round's
  // length (its row tiles, and the weights' way from L2 and the ends as one more)
  int best = 8;
  int64_t best_t = INT64_MAX;
  for (int rt : {8, 7, 6, 4, 2}) {
    const int64_t blocks = (a.R + 16 * rt - 1) / (16 * rt), t = (blocks + 255) / 256 * (rt + 1);
    if (t < best_t) {
      best_t = t;
      best = rt;
    }
  }
  switch (best) {
    case 8: return launch_rt<8>(a, s);
    case 7: return launch_rt<7>(a, s);
    case 6: return launch_rt<6>(a, s);
    case 4: return launch_rt<4>(a, s);
    default: return launch_rt<2>(a, s);
  }
}

}  // namespace ivhd
