// Device helpers shared by the kernels of drot_kernels.hip and
// drot_resident.h: wave-level sums, memory helpers, and the scalar steps that
// close an iteration.
#pragma once

#include <type_traits>

#include "drot_internal.h"

namespace drot {
namespace {

// ---------------------------------------------------------------------------
// Wave-level sum with DPP (all 64 lanes active).  Fixed combination order;
// the result is read from lane 63.
// ---------------------------------------------------------------------------
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}

template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, dpp_i<CTRL, ROW_MASK>(__builtin_bit_cast(int, v)));
}

template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ double dpp(double v) {
  const unsigned long long bits = __builtin_bit_cast(unsigned long long, v);
  const int lo = dpp_i<CTRL, ROW_MASK>((int)(unsigned)(bits & 0xffffffffull));
  const int hi = dpp_i<CTRL, ROW_MASK>((int)(unsigned)(bits >> 32));
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

__device__ __forceinline__ float lane63(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

__device__ __forceinline__ double lane63(double v) {
  const unsigned long long bits = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)(bits & 0xffffffffull), 63);
  const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(bits >> 32), 63);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

template <typename V>
__device__ __forceinline__ V wave_sum(V v) {
  v += dpp<0xB1>(v);         // quad_perm [1,0,3,2]: pairs
  v += dpp<0x4E>(v);         // quad_perm [2,3,0,1]: quads
  v += dpp<0x141>(v);        // row_half_mirror: groups of 8
  v += dpp<0x140>(v);        // row_mirror: rows of 16
  v += dpp<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
  return lane63(v);
}

__device__ __forceinline__ double read_lane(double v, int l) {
  const unsigned long long bits = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)(bits & 0xffffffffull), l);
  const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(bits >> 32), l);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// wave_sum of N values at once: each DPP step is applied to all N before the
// next, so that the N dependency chains overlap.  Every lane gets the totals.
template <int N>
__device__ __forceinline__ void wave_sum_n(double (&v)[N]) {
#pragma unroll
  for (int s = 0; s < N; ++s) v[s] += dpp<0xB1>(v[s]);
#pragma unroll
  for (int s = 0; s < N; ++s) v[s] += dpp<0x4E>(v[s]);
#pragma unroll
  for (int s = 0; s < N; ++s) v[s] += dpp<0x141>(v[s]);
#pragma unroll
  for (int s = 0; s < N; ++s) v[s] += dpp<0x140>(v[s]);
#pragma unroll
  for (int s = 0; s < N; ++s) v[s] += dpp<0x142, 0xA>(v[s]);
#pragma unroll
  for (int s = 0; s < N; ++s) v[s] += dpp<0x143, 0xC>(v[s]);
#pragma unroll
  for (int s = 0; s < N; ++s) v[s] = lane63(v[s]);
}

// Lanes l < 32 get a's two halves added, lanes l >= 32 b's (v_permlane32_swap),
// and the same for the even and odd rows of 16 lanes (v_permlane16_swap).
__device__ __forceinline__ void swap32(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a),
                                                  __builtin_bit_cast(uint32_t, b), false, false);
  a = __builtin_bit_cast(float, (uint32_t)r[0]);
  b = __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ void swap16(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a),
                                                  __builtin_bit_cast(uint32_t, b), false, false);
  a = __builtin_bit_cast(float, (uint32_t)r[0]);
  b = __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ void swap32(double& a, double& b) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  a = __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi[0] << 32) | (uint32_t)lo[0]);
  b = __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi[1] << 32) | (uint32_t)lo[1]);
}
__device__ __forceinline__ void swap16(double& a, double& b) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  a = __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi[0] << 32) | (uint32_t)lo[0]);
  b = __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi[1] << 32) | (uint32_t)lo[1]);
}
template <typename V>
__device__ __forceinline__ V fold32(V a, V b) {
  swap32(a, b);
  return a + b;
}
template <typename V>
__device__ __forceinline__ V fold16(V a, V b) {
  swap16(a, b);
  return a + b;
}

// x / d with r = 1 / d at hand: one Newton step on the quotient, three
// operations in a row instead of the fifteen of a division.
__device__ __forceinline__ double div_by(double x, double d, double r) {
  const double q = x * r;
  return __builtin_fma(__builtin_fma(-d, q, x), r, q);
}

__device__ __forceinline__ float relu_of(float v) { return __builtin_fmaxf(v, 0.f); }
__device__ __forceinline__ double relu_of(double v) { return __builtin_fmax(v, 0.0); }

// ---------------------------------------------------------------------------
// Types and memory helpers.
// ---------------------------------------------------------------------------
// Partial sums of the float32 iteration are float32 (per tile); everything
// else accumulates in float64.
constexpr bool is_iter(int mode) { return mode == kIter || mode == kIterA || mode == kIterB; }
constexpr bool is_final(int mode) { return mode == kFinal || mode == kFinalW; }

template <typename T, int MODE>
struct PartialOf {
  using type = typename std::conditional<std::is_same<T, float>::value && is_iter(MODE), float,
                                         double>::type;
};

// rho * c rounded once (never fused into a neighbouring add), so that the
// skip-C schedule's W = X - rho C and its restoration X = W + rho C use the
// same product and zero entries come back exactly zero.
template <typename A>
__device__ __forceinline__ A mul_rounded(A a, A b) {
#pragma clang fp contract(off)
  return a * b;
}

template <typename T, int VEC>
struct VecOf;
template <>
struct VecOf<float, 4> {
  typedef float type __attribute__((ext_vector_type(4)));
};
template <>
struct VecOf<double, 2> {
  typedef double type __attribute__((ext_vector_type(2)));
};

// 16-byte (or scalar) loads and stores; NT selects the nontemporal
// (streaming) cache policy, used when the plan and the cost matrix do not fit
// in the last-level cache.
template <typename T, int VEC, bool NT>
__device__ __forceinline__ void load_chunk(const T* ptr, T (&out)[VEC]) {
  if constexpr (VEC == 1) {
    out[0] = NT ? __builtin_nontemporal_load(ptr) : *ptr;
  } else {
    using V = typename VecOf<T, VEC>::type;
    const V* vp = reinterpret_cast<const V*>(ptr);
    const V v = NT ? __builtin_nontemporal_load(vp) : *vp;
#pragma unroll
    for (int e = 0; e < VEC; ++e) out[e] = v[e];
  }
}

template <typename T, int VEC, bool NT>
__device__ __forceinline__ void store_chunk(T* ptr, const T (&in)[VEC]) {
  if constexpr (VEC == 1) {
    if (NT) __builtin_nontemporal_store(in[0], ptr);
    else *ptr = in[0];
  } else {
    using V = typename VecOf<T, VEC>::type;
    V v;
#pragma unroll
    for (int e = 0; e < VEC; ++e) v[e] = in[e];
    if (NT) __builtin_nontemporal_store(v, reinterpret_cast<V*>(ptr));
    else *reinterpret_cast<V*>(ptr) = v;
  }
}

// VEC bfloat16 values (raw 16-bit patterns) widened exactly to float.
template <int VEC, bool NT>
__device__ __forceinline__ void load_bf16(const uint16_t* ptr, float (&out)[VEC]) {
  if constexpr (VEC == 1) {
    const uint16_t b = NT ? __builtin_nontemporal_load(ptr) : *ptr;
    out[0] = __builtin_bit_cast(float, (uint32_t)b << 16);
  } else {
    static_assert(VEC == 4, "bfloat16 chunks are 4 wide");
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    const u2* vp = reinterpret_cast<const u2*>(ptr);
    const u2 v = NT ? __builtin_nontemporal_load(vp) : *vp;
    out[0] = __builtin_bit_cast(float, v[0] << 16);
    out[1] = __builtin_bit_cast(float, v[0] & 0xffff0000u);
    out[2] = __builtin_bit_cast(float, v[1] << 16);
    out[3] = __builtin_bit_cast(float, v[1] & 0xffff0000u);
  }
}

__device__ __forceinline__ bool finite_d(double v) { return __builtin_isfinite(v); }

__device__ __forceinline__ void store_agent(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double load_agent(const double* p) {
  return __hip_atomic_load(const_cast<double*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The state scalars that the aux kernel and its finisher read.  Every
// workgroup loads them when it starts, so that the last workgroup's scalar
// steps wait on no further load; nothing in them changes during the launch
// (only the last workgroup writes the state, after all others are done).
// The value of one of two pointers, chosen by a wave-uniform condition.
// Each candidate is passed through readfirstlane first, so that the choice is
// made between values held in registers, never between addresses of
// argument fields (which would force the arguments into scratch memory).
template <typename P>
__device__ __forceinline__ P* pick(bool c, P* x, P* y) {
  auto uni = [](P* v) {
    const uint64_t u = reinterpret_cast<uint64_t>(v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return reinterpret_cast<P*>(((uint64_t)hi << 32) | lo);
  };
  const P* px = uni(x);
  const P* py = uni(y);
  return const_cast<P*>(c ? px : py);
}

struct StateIn {
  double rho, tol, alpha, sum_p, sum_q, norm_pq, norm_c;
  double cphi, cpsi, sum_phi0, sum_psi0;
  int64_t iter, max_iter;
  uint64_t t_start;
  int tol_mode, done;
};

__device__ __forceinline__ StateIn load_state(const DevState* st) {
  StateIn v;
  v.rho = st->rho;
  v.tol = st->tol;
  v.alpha = st->alpha;
  v.sum_p = st->sum_p;
  v.sum_q = st->sum_q;
  v.norm_pq = st->norm_pq;
  v.norm_c = st->norm_c;
  v.cphi = st->cphi;
  v.cpsi = st->cpsi;
  v.sum_phi0 = st->sum_phi0;
  v.sum_psi0 = st->sum_psi0;
  v.iter = st->iter;
  v.max_iter = st->max_iter;
  v.t_start = st->t_start;
  v.tol_mode = st->tol_mode;
  v.done = st->done;
  return v;
}

// The eight sums that close an iteration -- sum r, sum r^2, sum p phi~,
// sum s, sum s^2, sum q psi~, <C, X> and sum [t]_+^2 -- from the aux
// workgroups' published partials `bp` (slot-major [kSlots][nb]): each lane
// adds a fixed subset in a fixed order, then a DPP reduction; every lane of
// the wave gets the totals.  A column workgroup fills only the column and
// tile slots and a row workgroup the row and tile slots, and the sum skips
// the others.  AGENT: the sums were published by workgroups of the same
// launch (device-scope loads after the acquire fence); otherwise by an
// earlier launch, whose end made them visible to plain (cached) loads.
template <bool AGENT>
__device__ __forceinline__ void iter_sums(const double* bp, int nb, int col_wgs, double (&w)[8]) {
  constexpr int B = 4;  // workgroups per lane in flight
  const int lane = threadIdx.x & (kWave - 1);
  constexpr int slot[8] = {kSR, kSR2, kSPphi, kSS, kSS2, kSQpsi, kST0, kST1};
#pragma unroll
  for (int s = 0; s < 8; ++s) w[s] = 0.0;
  for (int k0 = 0; k0 < nb; k0 += B * kWave) {
    double v[B][8];
#pragma unroll
    for (int u = 0; u < B; ++u) {
#pragma unroll
      for (int s = 0; s < 8; ++s) v[u][s] = 0.0;
      if (k0 + u * kWave >= nb) continue;  // wave-uniform: no load in this block
      const int k = k0 + u * kWave + lane;
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        bool use = k < nb;
        if (s < 3) use = use && k >= col_wgs;
        else if (s < 6) use = use && k < col_wgs;
        const double* ptr = bp + (int64_t)slot[s] * nb + k;
        if (use) v[u][s] = AGENT ? load_agent(ptr) : *ptr;
      }
    }
#pragma unroll
    for (int u = 0; u < B; ++u)
#pragma unroll
      for (int s = 0; s < 8; ++s) w[s] += v[u][s];
  }
  wave_sum_n(w);
}

// The scalar steps closing iteration k = sv.iter + 1 (Algorithm 1 steps
// 5-8, scalar part, and the stopping criteria of Section 3) from the sums w
// of iter_sums and the state sv entering it: beta = f^T r / (m+n), the common
// scalar part 2 beta - alpha of the new shifts, alpha <- alpha - beta, the
// objectives, residuals and the test.  `nc`: the iteration read no C (the
// C-free step of the skip-C schedule), so it has no <C,X> and no dual
// residual: it records NaN for them and can only stop at max_iter.
struct ScalarStep {
  double cphi, cpsi, alpha, pobj, dobj, rp, rd, gap, test;
  int64_t k;
  int done, status;
};

// The objectives, residuals and the stopping test of iteration f.k, from its
// sums `w` and the shift parts f.cphi, f.cpsi and f.alpha it ends with.
__device__ __forceinline__ void scalar_tests(ScalarStep& f, const StateIn& sv,
                                             const double (&w)[8], bool nc) {
  const double rho = sv.rho;
  const double nan = __builtin_nan("");
  f.pobj = nc ? nan : w[6];
  f.dobj = (w[2] + f.cphi * sv.sum_p + w[5] + f.cpsi * sv.sum_q) / rho;
  f.gap = fabs(f.pobj - f.dobj);
  f.rp = sqrt(w[1] + w[4]);
  f.rd = nc ? nan : sqrt(w[7]) / rho;
  const double ep = f.rp / fmax(sv.norm_pq, 1e-300);
  const double ed = f.rd / fmax(sv.norm_c, 1e-300);
  const double eg = f.gap / fmax(fmax(fabs(f.pobj), fabs(f.dobj)), 1e-300);
  f.test = sv.tol_mode ? fmax(f.rp, fmax(f.rd, f.gap)) : fmax(ep, fmax(ed, eg));
  f.done = 0;
  f.status = 0;
  if ((!nc && !finite_d(f.test)) || !finite_d(f.alpha) || !finite_d(f.cphi) || !finite_d(f.rp)) {
    f.done = 1;
    f.status = -3;
  } else if (!nc && f.test <= sv.tol) {
    f.done = 1;
  } else if (f.k >= sv.max_iter) {
    f.done = 1;
    f.status = 1;
  }
}

__device__ __forceinline__ ScalarStep scalar_step(const StateIn& sv, const double (&w)[8],
                                                  int64_t m, int64_t n, bool nc) {
  ScalarStep f;
  const double mn = (double)(m + n);
  const double beta = w[0] / mn;
  const double cc = 2.0 * beta - sv.alpha;
  f.cphi = cc / (double)n;
  f.cpsi = cc / (double)m;
  f.alpha = sv.alpha - beta;
  f.k = sv.iter + 1;
  scalar_tests(f, sv, w, nc);
  return f;
}

// The trace record of iteration f.k into `tr`.  One thread.
__device__ __forceinline__ void trace_record(double* tr, const ScalarStep& f, uint64_t t_start,
                                             uint64_t now, double wall_rate) {
  tr[0] = f.pobj;
  tr[1] = f.dobj;
  tr[2] = f.rp;
  tr[3] = f.rd;
  tr[4] = f.gap;
  tr[5] = f.test;
  tr[6] = (double)(now - t_start) / wall_rate;
  tr[7] = (double)f.k;
}

// Write the state after iteration f.k into `dst` (a copy of `src`, the
// record entering it, with the iteration fields replaced) and its trace
// record.  One thread.
__device__ __forceinline__ void commit_step(DevState* dst, const DevState* src,
                                            const ScalarStep& f, const SweepArgs& a,
                                            uint64_t t_start) {
  const uint64_t now = wall_clock64();
  if (dst != src) *dst = *src;
  dst->alpha = f.alpha;
  dst->cphi = f.cphi;
  dst->cpsi = f.cpsi;
  dst->iter = f.k;
  dst->t_last = now;
  dst->pobj = f.pobj;
  dst->dobj = f.dobj;
  dst->rp = f.rp;
  dst->rd = f.rd;
  dst->gap = f.gap;
  dst->test = f.test;
  const int64_t slot = f.k - 1 < a.trace_cap ? f.k - 1 : (f.k - 1) % a.trace_cap;
  trace_record(a.trace + slot * kTraceWidth, f, t_start, now, a.wall_rate);
  if (f.done) {
    dst->done = 1;
    dst->status = f.status;
    dst->stop_iter = f.k;
    dst->t_stop = now;
  }
}

}  // namespace
}  // namespace drot
