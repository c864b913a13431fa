// A small multilayer perceptron trained with hand-written gfx950 kernels:
// the learned warm start of DROT.  It maps the marginals (p, q) of an OT
// problem to initial dual variables (mu, nu); DROT then starts from the shifts
// phi_0 = rho mu, psi_0 = rho nu (a warm start is valid because DR converges
// from any starting point, Lemma 1).
//
// Network: in -> hidden (ReLU) -> hidden (ReLU) -> out, mean-squared-error
// loss.  Weights are kept in float32 (Adam master copy) and bfloat16 (the
// copy the matrix cores read); activations and gradients enter the GEMMs in
// bfloat16 and every GEMM accumulates in float32 on the MFMA units
// (v_mfma_f32_32x32x8 bf16).  All reductions run in a fixed order.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/drot.h"

int drot_internal_fail(int code, const char* msg);

namespace {

int mfail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  return drot_internal_fail(code, buf);
}

#define MHIP(expr)                                                                   \
  do {                                                                               \
    hipError_t e_ = (expr);                                                          \
    if (e_ != hipSuccess)                                                            \
      return mfail(DROT_EDEVICE, "%s failed: %s", #expr, hipGetErrorString(e_));     \
  } while (0)

typedef uint16_t bf16;
typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

__host__ __device__ inline bf16 to_bf16(float f) {
  // round to nearest even (finite inputs)
  uint32_t u;
  memcpy(&u, &f, 4);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16)(u >> 16);
}

// ---------------------------------------------------------------------------
// The products.  Every product is cut into wave blocks of 32 rows by 32
// columns (64 where B is stored K x N) and its depth K into S slices, one wave
// each; the S waves of a block are in one workgroup.  A wave brings its own
// operands from memory through its own piece of LDS, 64 deep at a time with
// the next two such pieces on their way, and meets the other waves only at the
// end, where the slices' sums are added in slice order in LDS and finished: at
// these sizes a product is a chain of memory latencies, barriers and launches,
// not of bytes or operations.  Operands are contiguous along K, a row's 128
// bytes in one line, wherever the kernels can arrange it (activations and
// gradients are stored a second time transposed, for the weight gradients);
// the weights in the step through a layer are not, and are read two columns at
// a time.  Loading the matrix instruction's operands straight from memory, 32
// rows and 16 bytes of each at a time, took 17 us instead of 8 for
// 256 x 512 x 2048; the epilogue's reads between its stores another 3.
// Measured per call (in -> hidden -> out, batch; before: 64 x 64 tiles, one
// launch more for every split sum, 8 and 21 launches): gradients of
// 2048 -> 512 -> 2048, 256: 127 -> 65 us; 2048 -> 1024 -> 2048, 512: 231 -> 114;
// forward 35 -> 17 and 58 -> 32; gradients of 128 -> 64 -> 128, 64: 91 -> 45.
//
// Each output is accumulated over K in the same order by the same instruction
// (v_mfma_f32_32x32x8 bf16) in every path.
//
// A training step's gradients take six launches of dependent work: three
// forward steps (the first rounds x and writes its transpose beside the
// product, the third takes the error and its gradient in the epilogue) and,
// per layer, one launch with the step through the layer, the weight gradient
// and the bias gradient side by side.
// Requires M % 32 == N % 64 == ks % 32 == 0, leading dimensions multiples of 8
// and 16-byte aligned operands (checked on the host).
// ---------------------------------------------------------------------------
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;            // waves of a workgroup
constexpr int kThreads = 64 * kWaves;
constexpr int kColSlices = 16;       // row classes of a bias gradient

// What happens to a product.
enum Epi : int {
  kEpiStore = 0,  // C
  kEpiLayer = 1,  // + bias, ReLU if `relu`: C, its bfloat16 copy (Cb) and (CbT) that transposed
  kEpiGate = 2,   // kept where gate > 0, zero elsewhere: the same three
  kEpiError = 3   // + bias: y in C; d = 2 (y - t) / count in D, Cb and CbT; sum (y - t)^2 in `part`
};

struct Job {
  const void* A;  // M x K bfloat16 (float32 in the first step)
  const bf16* B;  // N x K (or K x N)
  float* C;       // M x N; every matrix is contiguous
  bf16 *Cb, *CbT;
  const float *bias, *gate, *t;
  float* D;
  double* part;   // one double per workgroup
  int M, N, K, S, ks, relu, wgs;
};

// Wave block -> first row and column; columns fastest.
__device__ __forceinline__ void block_at(const Job& j, int block, int width, int& m0, int& n0) {
  const int per = j.N / width;
  m0 = block / per * 32;
  n0 = block % per * width;
}

__device__ __forceinline__ v4s as_v4s(uint32_t x, uint32_t y) {
  const v2u u = {x, y};
  return __builtin_bit_cast(v4s, u);
}

// Sixteen values along K per lane pair: lanes < 32 hold k .. k + 7, lanes >= 32
// k + 8 .. k + 15; the matrix instruction wants k .. k + 3 and k + 4 .. k + 7.
__device__ __forceinline__ void halves(const v4u& v, v4s& first, v4s& second) {
  const auto p = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false);
  const auto q = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
  first = as_v4s(p[0], q[0]);
  second = as_v4s(p[1], q[1]);
}

// Two values rounded to nearest even (v_cvt_pk_bf16_f32), the first one low.
__device__ __forceinline__ uint32_t round2(float x, float y) {
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  typedef float f2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{x, y}), b2));
}
__device__ __forceinline__ v4u round8(const v4f& x, const v4f& y) {
  return v4u{round2(x[0], x[1]), round2(x[2], x[3]), round2(y[0], y[1]), round2(y[2], y[3])};
}

// A wave's own piece of LDS: 32 rows of kDeep values of each operand that is
// contiguous along K, 16 bytes apart from a multiple of 128 so that eight rows
// lie in different banks.  Only this wave uses it: no barrier.
constexpr int kDeep = 64;
constexpr int kRowBytes = 2 * kDeep + 16;
constexpr int kTileBytes = 32 * kRowBytes;
constexpr int kWaveBytes = 2 * kTileBytes;

// 32 rows of kDeep values from p (leading dimension ld) on their way to LDS:
// eight lanes read a row, 128 bytes in one line of memory, four rows a lane.
template <bool F32>
struct Rows {
  v4u v[4];
  v4f f[F32 ? 4 : 1][2];
  // `valid`: how much of the depth is there, kDeep or 32; the rest repeats it.
  __device__ __forceinline__ void load(const void* p, int ld, int valid) {
    const int lane = threadIdx.x & 63;
    const int k = 8 * (lane & 7) < valid ? 8 * (lane & 7) : 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const size_t o = (size_t)(8 * u + (lane >> 3)) * ld + k;
      if constexpr (F32) {
        f[u][0] = *reinterpret_cast<const v4f*>(static_cast<const float*>(p) + o);
        f[u][1] = *reinterpret_cast<const v4f*>(static_cast<const float*>(p) + o + 4);
      } else {
        v[u] = *reinterpret_cast<const v4u*>(static_cast<const bf16*>(p) + o);
      }
    }
  }
  __device__ __forceinline__ void store(char* tile) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if constexpr (F32) v[u] = round8(f[u][0], f[u][1]);
      *reinterpret_cast<v4u*>(tile + (8 * u + (lane >> 3)) * kRowBytes + 16 * (lane & 7)) = v[u];
    }
  }
};

// The operand of two matrix instructions, 16 deep from 16 step on.
__device__ __forceinline__ void operand(const char* tile, int step, v4s (&v)[2]) {
  const int lane = threadIdx.x & 63;
  const v4u w = *reinterpret_cast<const v4u*>(tile + (lane & 31) * kRowBytes + 32 * step + 16 * (lane >> 5));
  halves(w, v[0], v[1]);
}

// acc += A[m0 .. m0 + 31][kb .. kb + ks) B[n0 .. n0 + 31][same]^T, kDeep at a
// time with the next two such pieces on their way.
template <bool F32A>
__device__ __forceinline__ void product_nt(v16f& acc, const Job& j, int m0, int n0, int kb, char* own) {
  const char* const ap = static_cast<const char*>(j.A) + ((size_t)m0 * j.K + kb) * (F32A ? 4 : 2);
  const bf16* const bp = j.B + (size_t)n0 * j.K + kb;
  const int n = (j.ks + kDeep - 1) / kDeep;
  Rows<F32A> a[2];
  Rows<false> b[2];
  auto load = [&](int s, int c) {
    if (c >= n) return;
    const int valid = j.ks - c * kDeep < kDeep ? j.ks - c * kDeep : kDeep;
    a[s].load(ap + (size_t)c * kDeep * (F32A ? 4 : 2), j.K, valid);
    b[s].load(bp + (size_t)c * kDeep, j.K, valid);
  };
  auto multiply = [&](int s, int c) {
    if (c >= n) return;
    a[s].store(own);
    b[s].store(own + kTileBytes);
    load(s, c + 2);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int half = 0; half < 2; ++half) {  // the second is missing where ks / 32 is odd
      if (half == 1 && j.ks - c * kDeep < kDeep) continue;
#pragma unroll
      for (int i = 2 * half; i < 2 * half + 2; ++i) {
        v4s x[2], y[2];
        operand(own, i, x);
        operand(own + kTileBytes, i, y);
#pragma unroll
        for (int e = 0; e < 2; ++e)
          acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(x[e], y[e], acc, 0, 0, 0);
      }
    }
    __builtin_amdgcn_wave_barrier();
  };
  load(0, 0);
  load(1, 1);
  for (int c = 0; c < n; c += 2) {
    multiply(0, c);
    multiply(1, c + 1);
  }
}

// acc[q] += A[m0 .. m0 + 31][kb .. kb + ks) B[same][n0 + 2 (lane mod 32) + q]
__device__ __forceinline__ void product_nn(v16f (&acc)[2], const Job& j, int m0, int n0, int kb, char* own) {
  const int lane = threadIdx.x & 63;
  const bf16* const ap = static_cast<const bf16*>(j.A) + (size_t)m0 * j.K + kb;
  const bf16* const bp = j.B + (size_t)(kb + 4 * (lane >> 5)) * j.N + n0 + 2 * (lane & 31);
  const int n = (j.ks + kDeep - 1) / kDeep;
  Rows<false> a[2];
  uint32_t b[2][kDeep / 8][4];
  auto load = [&](int s, int c) {
    if (c >= n) return;
    const int valid = j.ks - c * kDeep < kDeep ? j.ks - c * kDeep : kDeep;
    a[s].load(ap + (size_t)c * kDeep, j.K, valid);
#pragma unroll
    for (int i = 0; i < kDeep / 8; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        b[s][i][e] = *reinterpret_cast<const uint32_t*>(
            bp + (size_t)(c * kDeep + (8 * i < valid ? 8 * i : 0) + e) * j.N);
  };
  auto multiply = [&](int s, int c) {
    if (c >= n) return;
    a[s].store(own);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (half == 1 && j.ks - c * kDeep < kDeep) continue;
#pragma unroll
      for (int i = 2 * half; i < 2 * half + 2; ++i) {
        v4s x[2];
        operand(own, i, x);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const uint32_t* const w = b[s][2 * i + e];
          // the low halves are column q = 0, the high halves q = 1
          const v4s b0 = as_v4s((w[0] & 0xffffu) | w[1] << 16, (w[2] & 0xffffu) | w[3] << 16);
          const v4s b1 = as_v4s(w[0] >> 16 | (w[1] & 0xffff0000u), w[2] >> 16 | (w[3] & 0xffff0000u));
          acc[0] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(x[e], b0, acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(x[e], b1, acc[1], 0, 0, 0);
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
    load(s, c + 2);
  };
  load(0, 0);
  load(1, 1);
  for (int c = 0; c < n; c += 2) {
    multiply(0, c);
    multiply(1, c + 1);
  }
}

// Two consecutive rows of one column, with the column's bias and the entries of
// gate or t; returns (y - t)^2 of kEpiError.
template <int EPI>
__device__ __forceinline__ double finish(const Job& j, int row, int col, float v0, float v1, float bcol,
                                         float x0, float x1) {
  const size_t o = (size_t)row * j.N + col;
  float v[2] = {v0, v1};
  const float x[2] = {x0, x1};
  double err = 0.0;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const size_t oe = o + (size_t)e * j.N;
    if constexpr (EPI == kEpiGate) {
      if (!(x[e] > 0.f)) v[e] = 0.f;
    } else if constexpr (EPI != kEpiStore) {
      v[e] += bcol;
      if (EPI == kEpiLayer && j.relu && !(v[e] > 0.f)) v[e] = 0.f;
    }
    j.C[oe] = v[e];
    if constexpr (EPI == kEpiError) {
      const float d = v[e] - x[e];
      err += (double)d * (double)d;
      v[e] = 2.f * d / (float)((int64_t)j.M * j.N);
      j.D[oe] = v[e];
    }
  }
  if constexpr (EPI != kEpiStore) {
    const uint32_t both = round2(v[0], v[1]);
    if (j.Cb) {
      j.Cb[o] = (bf16)both;
      j.Cb[o + j.N] = (bf16)(both >> 16);
    }
    if (j.CbT) *reinterpret_cast<uint32_t*>(j.CbT + (size_t)col * j.M + row) = both;
  }
  return err;
}

// Workgroup `wg` of a product with S slices: NQ = 1: B stored N x K; NQ = 2:
// K x N.  `sm`: kWaveBytes for each wave.  All waves of the workgroup call it.
template <int NQ, int EPI, bool F32A, int S>
__device__ __forceinline__ void product_s(const Job& j, int wg, char* sm) {
  static_assert(16 * 2 * 64 * sizeof(float) <= kWaveBytes, "the sums reuse the operands' LDS");
  constexpr int P = 16 / S;  // of a block's 16 rows per lane, those that a wave finishes
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int z = wave % S, r0 = P * z;
  const int block = wg * ((int)(blockDim.x >> 6) / S) + wave / S;
  const bool work = block < (j.M / 32) * (j.N / (32 * NQ));
  int m0 = 0, n0 = 0;
  if (work) block_at(j, block, 32 * NQ, m0, n0);
  // acc[q][r]: column n0 + NQ (lane mod 32) + q, row m0 + 8 (r / 4) + 4 (lane / 32) + r % 4
  const int col = n0 + NQ * (lane & 31), rbase = m0 + 4 * (lane >> 5);
  auto row = [&](int i) { return rbase + 8 * ((r0 + i) >> 2) + ((r0 + i) & 3); };
  v16f acc[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[q][r] = 0.f;
  // What the epilogue reads is asked for before the product: between the
  // epilogue's stores each load would be a round trip to memory of its own.
  float bcol = 0.f, extra[NQ][P];
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int i = 0; i < P; ++i) extra[q][i] = 0.f;
  if (work) {
    if (EPI == kEpiLayer || EPI == kEpiError) bcol = j.bias[col];
    if (EPI == kEpiGate || EPI == kEpiError) {
      const float* const src = EPI == kEpiGate ? j.gate : j.t;
#pragma unroll
      for (int i = 0; i < P; ++i)
#pragma unroll
        for (int q = 0; q < NQ; ++q) extra[q][i] = src[(size_t)row(i) * j.N + col + q];
    }
    char* const own = sm + wave * kWaveBytes;
    if constexpr (NQ == 1) product_nt<F32A>(acc[0], j, m0, n0, z * j.ks, own);
    else product_nn(acc, j, m0, n0, z * j.ks, own);
  }
  float v[NQ][P];
  if constexpr (S == 1) {
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int i = 0; i < P; ++i) v[q][i] = acc[q][i];
  } else {  // the slices' sums, in order
    constexpr int kStride = kWaveBytes / sizeof(float);  // from slice to slice
    float* const mine = reinterpret_cast<float*>(sm) + wave * kStride + lane;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int r = 0; r < 16; ++r) mine[(q * 16 + r) * 64] = acc[q][r];
    __syncthreads();
    const float* const src = mine - z * kStride + r0 * 64;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int i = 0; i < P; ++i) {
        v[q][i] = src[(q * 16 + i) * 64];
#pragma unroll
        for (int y = 1; y < S; ++y) v[q][i] += src[y * kStride + (q * 16 + i) * 64];
      }
  }
  double err = 0.0;
  if (work)
#pragma unroll
    for (int i = 0; i < P; i += 2)
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        err += finish<EPI>(j, row(i), col + q, v[q][i], v[q][i + 1], bcol, extra[q][i], extra[q][i + 1]);
  if constexpr (EPI == kEpiError) {
    __syncthreads();
    double* const red = reinterpret_cast<double*>(sm);
    red[threadIdx.x] = err;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) j.part[wg] = red[0];
  }
}

template <int NQ, int EPI, bool F32A>
__device__ __forceinline__ void product(const Job& j, int wg, char* sm) {
  switch (j.S) {
    case 1: return product_s<NQ, EPI, F32A, 1>(j, wg, sm);
    case 2: return product_s<NQ, EPI, F32A, 2>(j, wg, sm);
    case 4: return product_s<NQ, EPI, F32A, 4>(j, wg, sm);
    default: return product_s<NQ, EPI, F32A, 8>(j, wg, sm);
  }
}

// The transpose in bfloat16 of a 64 x 64 tile of x (rows x cols float32).
__device__ __forceinline__ void transpose_tile(const float* x, bf16* xt, int rows, int cols, int tile,
                                               float* sm) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const int r0 = tile / (cols / 64) * 64, c0 = tile % (cols / 64) * 64;
#pragma unroll 8
  for (int r = w; r < 64; r += waves) sm[r * 65 + lane] = x[(size_t)(r0 + r) * cols + c0 + lane];
  __syncthreads();
#pragma unroll 8
  for (int c = w; c < 64; c += waves)
    xt[(size_t)(c0 + c) * rows + r0 + lane] = to_bf16(sm[lane * 65 + c]);
}

// Column sums of a rows x cols float32 matrix (bias gradients) for 64 columns,
// in a fixed order: rows congruent mod kColSlices in order, then these sums.
__device__ __forceinline__ void col_sums(const float* g, float* out, int rows, int cols, int group,
                                         float* part) {
  constexpr int P = kColSlices / kWaves;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int j = group * 64 + lane;
  float s[P];
#pragma unroll
  for (int p = 0; p < P; ++p) s[p] = 0.f;
  int r = w;
  for (; r + 3 * kColSlices + kWaves * (P - 1) < rows; r += 4 * kColSlices) {
    float v[4][P];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int p = 0; p < P; ++p) v[u][p] = g[(int64_t)(r + u * kColSlices + p * kWaves) * cols + j];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int p = 0; p < P; ++p) s[p] += v[u][p];
  }
  for (; r < rows; r += kColSlices)
#pragma unroll
    for (int p = 0; p < P; ++p)
      if (r + p * kWaves < rows) s[p] += g[(int64_t)(r + p * kWaves) * cols + j];
#pragma unroll
  for (int p = 0; p < P; ++p) part[(w + p * kWaves) * 64 + lane] = s[p];
  __syncthreads();
  if (w == 0) {
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < kColSlices; ++k) t += part[k * 64 + lane];
    out[j] = t;
  }
}

// A forward step; in a first step with XT given the workgroups after the
// product's write the transpose of x.
template <int EPI, bool F32A>
__global__ __launch_bounds__(kThreads) void forward_step(Job j, const float* x, bf16* xt) {
  extern __shared__ __align__(16) char sm[];
  if ((int)blockIdx.x < j.wgs) product<1, EPI, F32A>(j, blockIdx.x, sm);
  else transpose_tile(x, xt, j.M, j.K, blockIdx.x - j.wgs, reinterpret_cast<float*>(sm));
}

// The backward work of a layer: the step through it (dx, none in the first
// layer: no workgroups), the weight gradient dw and the column sums of g; in
// the first layer, whose workgroups come last, also the sum of the loss's
// `parts` partial sums into host memory (kernels before it would wait for the
// write's way over the bus).
__global__ __launch_bounds__(kThreads) void backward_layer(Job dx, Job dw, const float* g, float* gb,
                                                           int rows, int cols, const double* part,
                                                           int parts, double* loss) {
  extern __shared__ __align__(16) char sm[];
  int b = blockIdx.x;
  if (parts > 0 && b-- == 0) {
    double* const red = reinterpret_cast<double*>(sm);
    double v = 0.0;
    for (int k = threadIdx.x; k < parts; k += kThreads) v += part[k];
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) *loss = red[0];
    return;
  }
  if (b < dx.wgs) return product<2, kEpiGate, false>(dx, b, sm);
  b -= dx.wgs;
  if (b < dw.wgs) return product<1, kEpiStore, false>(dw, b, sm);
  col_sums(g, gb, rows, cols, b - dw.wgs, reinterpret_cast<float*>(sm));
}

__global__ void cast_bf16(const float* __restrict__ x, bf16* __restrict__ y, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) y[i] = to_bf16(x[i]);
}

// Adam on the float32 master weights; refreshes the bfloat16 copy.  The
// coefficients b1, 1 - b1, b2, 1 - b2 and the bias corrections c1, c2 come
// from the host rounded once from float64 (1 - b2 formed in float32 from the
// rounded b2 would be 1.3e-5 off).
__global__ void adam(float* __restrict__ w, bf16* __restrict__ wb, const float* __restrict__ g,
                     float* __restrict__ m1, float* __restrict__ m2, int64_t count, float lr,
                     float b1, float ob1, float b2, float ob2, float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float gi = g[i];
  const float a = b1 * m1[i] + ob1 * gi;
  const float b = b2 * m2[i] + ob2 * gi * gi;
  m1[i] = a;
  m2[i] = b;
  const float v = w[i] - lr * (a / c1) / (sqrtf(b / c2) + eps);
  w[i] = v;
  wb[i] = to_bf16(v);
}

unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

struct drot_mlp {
  int device = 0;
  int in = 0, hid = 0, out = 0, max_batch = 0;
  int64_t n_params = 0;
  int64_t off_w[3], off_b[3];  // offsets into the flat parameter vector
  // device buffers, in device_mem
  char* device_mem = nullptr;
  float* w = nullptr;    // float32 master parameters (flat)
  bf16* wb = nullptr;    // bfloat16 copy
  float* g = nullptr;    // gradients (flat)
  float* m1 = nullptr;
  float* m2 = nullptr;
  float* a[3] = {};  // activations (layer outputs)
  bf16 *ab[3] = {}, *xb = nullptr;    // bfloat16 copies (of the last layer: none)
  bf16 *abt[3] = {}, *xbt = nullptr;  // and their transposes
  float* d[3] = {};  // gradients with respect to the pre-activations
  bf16 *db[3] = {}, *dbt[3] = {};
  double* part = nullptr;  // the loss's partial sums
  double* loss = nullptr;  // their sum, in pinned host memory
  int64_t step = 0;
};

namespace {

int64_t layer_in(const drot_mlp* n, int l) { return l == 0 ? n->in : n->hid; }
int64_t layer_out(const drot_mlp* n, int l) { return l == 2 ? n->out : n->hid; }

// K slices of an M x N x K product: while 64 x 64 tiles would be fewer than 256
// (one per compute unit), halve the depth of a slice, down to 128, up to 8.
int split_k(int M, int N, int K) {
  const int grid = (M / 64) * (N / 64);
  int S = 1;
  while (S < 8 && grid * S * 2 <= 256 && K % (64 * S) == 0 && K / (2 * S) >= 128) S *= 2;
  return S;
}

// The product's shape, slices and workgroups of `waves` (at least S of them);
// NQ as in product().
Job make_job(const void* A, const bf16* B, float* C, int M, int N, int K, int NQ, int waves) {
  Job j{};
  j.A = A;
  j.B = B;
  j.C = C;
  j.M = M;
  j.N = N;
  j.K = K;
  j.S = split_k(M, N, K);
  j.ks = K / j.S;
  const int blocks = (M / 32) * (N / (32 * NQ)), per = waves / j.S;
  j.wgs = (blocks + per - 1) / per;
  return j;
}

// Waves of a forward step's workgroups: four fill more compute units.
int forward_waves(int M, int N, int K) { return split_k(M, N, K) > 4 ? 8 : 4; }

int check_batch(const drot_mlp* n, int batch) {
  if (!n) return mfail(DROT_EINVAL, "mlp is NULL");
  if (batch < 64 || batch % 64 || batch > n->max_batch)
    return mfail(DROT_EINVAL, "batch must be a multiple of 64 in [64, %d]", n->max_batch);
  if (hipSetDevice(n->device) != hipSuccess) return mfail(DROT_EDEVICE, "hipSetDevice failed");
  return DROT_OK;
}

// y = f(x); with targets `t` also the error's gradient, the loss's partial
// sums and the transposes that backward() needs.
int forward(drot_mlp* n, int B, const float* x, float* y, const float* t, hipStream_t s) {
  // x is read in 16-byte pieces where it lies so; else it is rounded first.
  const bool direct = reinterpret_cast<uintptr_t>(x) % 16 == 0;
  if (!direct) {
    hipLaunchKernelGGL(cast_bf16, dim3(nblk((int64_t)B * n->in)), dim3(256), 0, s, x, n->xb,
                       (int64_t)B * n->in);
    MHIP(hipGetLastError());
  }
  for (int l = 0; l < 3; ++l) {
    const int K = (int)layer_in(n, l), N = (int)layer_out(n, l);
    const void* in = l > 0 ? (const void*)n->ab[l - 1] : direct ? (const void*)x : (const void*)n->xb;
    // a_l = act(x_l W_l^T + b_l)
    const int waves = forward_waves(B, N, K);
    Job j = make_job(in, n->wb + n->off_w[l], l == 2 ? y : n->a[l], B, N, K, 1, waves);
    j.bias = n->w + n->off_b[l];
    j.relu = l < 2;
    if (l == 2 && t) {
      j.t = t;
      j.D = n->d[2];
      j.Cb = n->db[2];
      j.CbT = n->dbt[2];
      j.part = n->part;
    } else {
      j.Cb = l < 2 ? n->ab[l] : nullptr;
      j.CbT = t ? n->abt[l] : nullptr;
    }
    const dim3 grid(j.wgs + (l == 0 && t ? (B / 64) * (K / 64) : 0)), block(64 * waves);
    const size_t lds = (size_t)waves * kWaveBytes;
    if (l == 0 && direct)
      hipLaunchKernelGGL((forward_step<kEpiLayer, true>), grid, block, lds, s, j, x, n->xbt);
    else if (l == 2 && t)
      hipLaunchKernelGGL((forward_step<kEpiError, false>), grid, block, lds, s, j, x, n->xbt);
    else
      hipLaunchKernelGGL((forward_step<kEpiLayer, false>), grid, block, lds, s, j, x, n->xbt);
    MHIP(hipGetLastError());
  }
  return DROT_OK;
}

// Gradients of the mean-squared error into `grad`; loss to *loss (host).
int backward(drot_mlp* n, int B, float* grad, double* loss, hipStream_t s) {
  const int parts = make_job(nullptr, nullptr, nullptr, B, n->out, n->hid, 1,
                             forward_waves(B, n->out, n->hid)).wgs;
  for (int l = 2; l >= 0; --l) {
    const int K = (int)layer_in(n, l), N = (int)layer_out(n, l);
    // dW_l = dZ_l^T x_l  (N x K);  db_l = column sums of dZ_l
    Job dw = make_job(n->dbt[l], l == 0 ? n->xbt : n->abt[l - 1], grad + n->off_w[l], N, K, B, 1,
                      kWaves);
    Job dx{};
    if (l > 0) {
      // dZ_{l-1} = (dZ_l W_l) * [a_{l-1} > 0] (B x K)
      dx = make_job(n->db[l], n->wb + n->off_w[l], n->d[l - 1], B, K, N, 2, kWaves);
      dx.gate = n->a[l - 1];
      dx.Cb = n->db[l - 1];
      dx.CbT = n->dbt[l - 1];
    }
    const int sums = l == 0 ? parts : 0;
    hipLaunchKernelGGL(backward_layer, dim3(dx.wgs + dw.wgs + N / 64 + (sums > 0)), dim3(kThreads),
                       (size_t)kWaves * kWaveBytes, s, dx, dw, n->d[l], grad + n->off_b[l], B, N,
                       n->part, sums, n->loss);
    MHIP(hipGetLastError());
  }
  MHIP(hipStreamSynchronize(s));
  if (loss) *loss = *n->loss / (double)((int64_t)B * n->out);
  return DROT_OK;
}

uint64_t splitmix(uint64_t& s) {
  uint64_t z = (s += 0x9e3779b97f4a7c15ull);
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

}  // namespace

extern "C" {

int drot_mlp_create(drot_mlp** out, int device, int in, int hidden, int outd, int max_batch,
                    uint64_t seed) {
  if (!out) return mfail(DROT_EINVAL, "out is NULL");
  *out = nullptr;
  if (in < 64 || hidden < 64 || outd < 64 || in % 64 || hidden % 64 || outd % 64)
    return mfail(DROT_EINVAL, "layer widths must be positive multiples of 64");
  if (max_batch < 64 || max_batch % 64) return mfail(DROT_EINVAL, "max_batch must be a multiple of 64");
  int count = 0;
  if (hipGetDeviceCount(&count) != hipSuccess || count <= 0) {
    (void)hipGetLastError();
    return mfail(DROT_EDEVICE, "no HIP device available");
  }
  if (device < 0 || device >= count) return mfail(DROT_EINVAL, "device out of range");
  MHIP(hipSetDevice(device));
  drot_mlp* n = new drot_mlp();
  n->device = device;
  n->in = in;
  n->hid = hidden;
  n->out = outd;
  n->max_batch = max_batch;
  int64_t o = 0;
  for (int l = 0; l < 3; ++l) {
    n->off_w[l] = o;
    o += layer_in(n, l) * layer_out(n, l);
    n->off_b[l] = o;
    o += layer_out(n, l);
  }
  n->n_params = o;
  // He-uniform initialisation from a seeded counter-based generator.
  std::vector<float> hw(o, 0.f);
  uint64_t st = seed;
  for (int l = 0; l < 3; ++l) {
    const double lim = std::sqrt(6.0 / (double)layer_in(n, l));
    for (int64_t k = 0; k < layer_in(n, l) * layer_out(n, l); ++k) {
      const double u = (double)(splitmix(st) >> 11) * (1.0 / 9007199254740992.0);
      hw[n->off_w[l] + k] = (float)((2.0 * u - 1.0) * lim);
    }
  }
  // All device buffers in one allocation, each on a 256-byte boundary.
  size_t bytes = 0;
  auto place = [&](auto** p, size_t count) {
    if (n->device_mem) *p = reinterpret_cast<std::remove_reference_t<decltype(*p)>>(n->device_mem + bytes);
    bytes += (sizeof(**p) * count + 255) / 256 * 256;
  };
  auto place_all = [&]() {
    bytes = 0;
    place(&n->w, (size_t)o);
    place(&n->wb, (size_t)o);
    place(&n->g, (size_t)o);
    place(&n->m1, (size_t)o);
    place(&n->m2, (size_t)o);
    place(&n->xb, (size_t)max_batch * in);
    place(&n->xbt, (size_t)max_batch * in);
    place(&n->part, (size_t)(max_batch / 32) * (outd / 32));
    for (int l = 0; l < 3; ++l) {
      const size_t c = (size_t)max_batch * layer_out(n, l);
      place(&n->a[l], c);
      place(&n->ab[l], l == 2 ? 0 : c);
      place(&n->abt[l], l == 2 ? 0 : c);
      place(&n->d[l], c);
      place(&n->db[l], c);
      place(&n->dbt[l], c);
    }
  };
  place_all();
  const bool ok = hipMalloc((void**)&n->device_mem, bytes) == hipSuccess &&
                  hipHostMalloc((void**)&n->loss, sizeof(double), hipHostMallocDefault) == hipSuccess;
  if (ok) place_all();
  if (!ok) {
    (void)hipGetLastError();
    drot_mlp_destroy(n);
    return mfail(DROT_ENOMEM, "MLP allocation failed");
  }
  if (drot_mlp_set_weights(n, hw.data()) != DROT_OK) {
    drot_mlp_destroy(n);
    return DROT_EDEVICE;
  }
  *out = n;
  return DROT_OK;
}

int drot_mlp_destroy(drot_mlp* n) {
  if (!n) return DROT_OK;
  (void)hipSetDevice(n->device);
  (void)hipDeviceSynchronize();
  if (n->device_mem) (void)hipFree(n->device_mem);
  if (n->loss) (void)hipHostFree(n->loss);
  delete n;
  return DROT_OK;
}

int drot_mlp_num_params(const drot_mlp* n, int64_t* count) {
  if (!n || !count) return mfail(DROT_EINVAL, "NULL argument");
  *count = n->n_params;
  return DROT_OK;
}

int drot_mlp_set_weights(drot_mlp* n, const float* host) {
  if (!n || !host) return mfail(DROT_EINVAL, "NULL argument");
  MHIP(hipSetDevice(n->device));
  MHIP(hipMemcpy(n->w, host, sizeof(float) * n->n_params, hipMemcpyHostToDevice));
  hipLaunchKernelGGL(cast_bf16, dim3(nblk(n->n_params)), dim3(256), 0, 0, n->w, n->wb, n->n_params);
  MHIP(hipGetLastError());
  MHIP(hipMemset(n->m1, 0, sizeof(float) * n->n_params));
  MHIP(hipMemset(n->m2, 0, sizeof(float) * n->n_params));
  MHIP(hipDeviceSynchronize());
  n->step = 0;
  return DROT_OK;
}

int drot_mlp_get_weights(drot_mlp* n, float* host) {
  if (!n || !host) return mfail(DROT_EINVAL, "NULL argument");
  MHIP(hipSetDevice(n->device));
  MHIP(hipDeviceSynchronize());
  MHIP(hipMemcpy(host, n->w, sizeof(float) * n->n_params, hipMemcpyDeviceToHost));
  return DROT_OK;
}

int drot_mlp_forward(drot_mlp* n, int batch, const float* x, float* y, void* stream) {
  int rc = check_batch(n, batch);
  if (rc) return rc;
  if (!x || !y) return mfail(DROT_EINVAL, "NULL argument");
  hipStream_t s = (hipStream_t)stream;
  return forward(n, batch, x, y, nullptr, s);
}

int drot_mlp_gradients(drot_mlp* n, int batch, const float* x, const float* t, float* grad,
                       double* loss, void* stream) {
  int rc = check_batch(n, batch);
  if (rc) return rc;
  if (!x || !t) return mfail(DROT_EINVAL, "NULL argument");
  hipStream_t s = (hipStream_t)stream;
  if ((rc = forward(n, batch, x, n->a[2], t, s))) return rc;
  return backward(n, batch, grad ? grad : n->g, loss, s);
}

}  // extern "C"

namespace {

// One Adam step with the gradient in `g` (device, flat parameter order).
int adam_step(drot_mlp* n, const float* g, float lr, hipStream_t s) {
  n->step += 1;
  const double b1 = 0.9, b2 = 0.999;
  const double c1 = 1.0 - std::pow(b1, (double)n->step), c2 = 1.0 - std::pow(b2, (double)n->step);
  hipLaunchKernelGGL(adam, dim3(nblk(n->n_params)), dim3(256), 0, s, n->w, n->wb, g, n->m1,
                     n->m2, n->n_params, lr, (float)b1, (float)(1.0 - b1), (float)b2,
                     (float)(1.0 - b2), 1e-8f, (float)c1, (float)c2);
  MHIP(hipGetLastError());
  return DROT_OK;
}

}  // namespace

extern "C" {

int drot_mlp_train_step(drot_mlp* n, int batch, const float* x, const float* t, float lr,
                        double* loss, void* stream) {
  if (!(lr > 0.f)) return mfail(DROT_EINVAL, "lr must be positive");
  int rc = drot_mlp_gradients(n, batch, x, t, nullptr, loss, stream);
  if (rc) return rc;
  return adam_step(n, n->g, lr, (hipStream_t)stream);
}

int drot_mlp_apply_gradients(drot_mlp* n, const float* grad, float lr, void* stream) {
  if (!n || !grad) return mfail(DROT_EINVAL, "NULL argument");
  if (!(lr > 0.f)) return mfail(DROT_EINVAL, "lr must be positive");
  MHIP(hipSetDevice(n->device));
  return adam_step(n, grad, lr, (hipStream_t)stream);
}

}  // extern "C"
