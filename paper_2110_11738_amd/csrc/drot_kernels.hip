// HIP kernels of the DROT hot path for gfx950 (CDNA4, wave64).
//
// One iteration of Algorithm 1 (DROT) is two launches:
//
//  sweep_kernel  one fused pass over the dense m x n plan.  Each entry is read
//                once (X and C) and written once (X):
//                    t     = phi_i + psi_j - rho c_ij
//                    x_ij <- max(x_ij + t, 0)                       (step 4)
//                and in the same pass the kernel accumulates row sums, column
//                sums (step 5), <C, X_{k+1}> and sum [t]_+^2 = rho^2 r_dual^2
//                at the incoming shifts (Section 3, stopping criteria), and
//                writes them as per-tile partials.
//  aux_kernel    the O(m+n) part: level-2 sums of the partials in a fixed
//                order; r = u - p, s = v - q; the vector parts of the new
//                shifts phi~ = (a - 2r)/n, psi~ = (b - 2s)/m; a <- a - r,
//                b <- b - s (steps 5-8).  The last workgroup to finish sums
//                the workgroups' scalar partials in a fixed order and does the
//                scalar steps: beta = f^T r/(m+n), the common scalar part
//                (2 beta - alpha) of the new shifts, alpha <- alpha - beta,
//                and the stopping test.  With many aux workgroups (and in the
//                batched solver) a separate one-wave finish_kernel does these
//                scalar steps instead, after the aux launch.
//
// The shifts are kept as phi = phi~ + (2 beta - alpha)/n and
// psi = psi~ + (2 beta - alpha)/m (the algebra of steps 6-7): the vector parts
// need no global quantity, and the next sweep adds the two scalar parts to its
// row shift, so no second pass over the vectors is needed once beta is known.
//
// Every sum runs in a fixed order, so results are bit-reproducible; the only
// atomics are the integer counter that elects the last aux workgroup and the
// maximum of the coordinates cost (order-independent).
//
// Differences from the paper's CUDA kernel (Section 3, "Main kernel"): that
// kernel is column-major with one thread per row and sums columns with float
// atomics.  Here X is row-major, the 64 lanes of a wavefront run along a row
// with 16-byte loads, each lane keeps the column partials of its columns in
// registers over the tile's rows, row sums use DPP cross-lane reductions, and
// column partials go through a deterministic two-level tree.  The kernel
// boundary between sweep and aux is the device-wide release/acquire point: a
// device-scope fence inside the sweep would write back the L2 (full of the
// freshly written plan) once per workgroup.
#include <hip/hip_ext.h>
#include <type_traits>

#include "drot_device.h"
#include "drot_internal.h"
#include "drot_small.h"

namespace drot {
namespace {

// Block-wide fixed-order sum of kSlots values; result valid in thread 0.
__device__ __forceinline__ void block_sum_slots(double (&acc)[kSlots],
                                                double (&red)[kSlots][kWaves]) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  __syncthreads();  // `red` may still be read from a previous use
#pragma unroll
  for (int s = 0; s < kSlots; ++s) {
    const double v = wave_sum(acc[s]);
    if (lane == 0) red[s][wave] = v;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
      double v = red[s][0];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) v += red[s][w];
      acc[s] = v;
    }
  }
}

// Run by one wave (all lanes active) once every aux workgroup's sums are in
// `bp`: the last aux workgroup, or a one-wave finishing launch.  Fixed-order
// sum of the workgroups' scalar partials, then, in lane 0, the scalar steps
// of the iteration (from the record `src`, committed to `dst`), of the
// initialisation or of the final evaluation (into `dst`).
template <int MODE>
__device__ void finish_global(const SweepArgs& a, const StateIn& sv, int nb, int col_wgs,
                              const DevState* src, const double* bp, DevState* dst) {
  const int lane = threadIdx.x;
  if (is_iter(MODE)) {
    double w[8];
    iter_sums<true>(bp, nb, col_wgs, w);
    if (lane != 0) return;
    const ScalarStep f = scalar_step(sv, w, a.g.m, a.g.n, MODE == kIterB);
    commit_step(dst, src, f, a, sv.t_start);
    return;
  }
  constexpr int B = 4;  // blockpart columns per lane in flight
  double acc[kSlots];
#pragma unroll
  for (int s = 0; s < kSlots; ++s) acc[s] = 0.0;
  for (int k0 = 0; k0 < nb; k0 += B * kWave) {
    double v[B][kSlots];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int k = k0 + u * kWave + lane;
#pragma unroll
      for (int s = 0; s < kSlots; ++s)
        v[u][s] = k < nb ? load_agent(bp + (int64_t)s * nb + k) : 0.0;
    }
#pragma unroll
    for (int u = 0; u < B; ++u)
#pragma unroll
      for (int s = 0; s < kSlots; ++s) acc[s] += v[u][s];
  }
  wave_sum_n(acc);
  if (lane != 0) return;

  DevState* st = dst;
  const int64_t m = a.g.m, n = a.g.n;
  const double mn = (double)(m + n);
  const double rho = sv.rho;
  const uint64_t now = wall_clock64();
  if (is_final(MODE)) {
    const double pobj = acc[kST0];
    const double dobj = (acc[kSPphi] + acc[kSQpsi]) / rho;
    st->f_pobj = pobj;
    st->f_dobj = dobj;
    st->f_rp = sqrt(acc[kSR2] + acc[kSS2]);
    st->f_rd = sqrt(acc[kST1]) / rho;
    st->f_gap = fabs(pobj - dobj);
    st->f_eps_p = st->f_rp / fmax(sv.norm_pq, 1e-300);
    st->f_eps_d = st->f_rd / fmax(sv.norm_c, 1e-300);
    st->f_eps_g = st->f_gap / fmax(fmax(fabs(pobj), fabs(dobj)), 1e-300);
  } else {
    st->alpha = acc[kSR] / mn;
    st->sum_p = acc[kSP];
    st->sum_q = acc[kSQ];
    st->norm_pq = sqrt(acc[kSPQ2]);
    st->norm_c = sqrt(acc[kST0]);
    st->init_bad = acc[kST1] + acc[kSNonfin];
    st->init_neg = acc[kSNeg];
    st->cphi = 0.0;
    st->cpsi = 0.0;
    st->iter = 0;
    st->done = 0;
    st->status = 0;
    st->stop_iter = 0;
    st->t_last = now;
  }
}

// Loads of a strided sequence (base[r * stride], r0 <= r < r1) added into
// `s` in ascending r, with the loads issued in masked batches of U so that a
// short sequence costs one memory latency.
template <int U, typename V, int CW>
__device__ __forceinline__ void sum_strided(const V* base, int64_t stride, int r0, int r1,
                                            double (&s)[CW]) {
  for (int rb = r0; rb < r1; rb += U) {
    V v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = rb + u;
      v[u] = r < r1 ? __builtin_nontemporal_load(base + (int64_t)r * stride) : V{};
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < CW; ++e) s[e] += (double)v[u][e];
  }
}

// ---------------------------------------------------------------------------
// The O(m+n) kernel.  Workgroups [0, col_wgs) own kAuxCols columns each: the
// column partials are read as 16-byte chunks with the row groups split over
// G thread groups, then combined in LDS in a fixed order.  The remaining
// workgroups own kAuxRows rows each, with the column strips' row partials
// split over the four waves.  All loads are issued up front, in masked
// batches, ahead of the stop flag's test.  Every scalar contribution (the
// per-column or per-row terms and a fixed slice of the tile scalars) lives in
// wave 0, which sums them with DPP, publishes them and takes part in the
// last-workgroup election; the other waves leave after the loads.  Wave 0 of
// the last workgroup does the scalar steps.
// ---------------------------------------------------------------------------
template <typename T, int MODE, bool WIDE = false, bool SPLIT = false>
__device__ __forceinline__ void aux_body(const SweepArgs& a, const int b, const int nb) {
  using P = typename std::conditional<WIDE, double, typename PartialOf<T, MODE>::type>::type;
  constexpr int CW = 16 / sizeof(P);      // columns per 16-byte chunk
  constexpr int NCH = kAuxCols / CW;      // chunks per workgroup
  constexpr int G = kBlock / NCH;         // row-group groups
  using V = typename VecOf<P, CW>::type;
  static_assert(G * kAuxCols >= kWaves * kAuxRows, "LDS buffer holds the row partials");
  static_assert(kAuxCols <= kWave && kAuxRows == kWave, "wave 0 finishes the entries");

  const StateIn sv = load_state(a.st);
  __shared__ double red2[G * kAuxCols];

  const int64_t m = a.g.m, n = a.g.n;
  const int col_wgs = (int)((n + kAuxCols - 1) / kAuxCols);
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const bool is_col = b < col_wgs;

  // Stage 1: loads.  `idx` is the column (column workgroups, threads below
  // kAuxCols) or row (row workgroups, wave 0) this thread finishes, else -1;
  // `w0`, `w1` its marginal entry and its accumulator (or phi / psi, or the
  // warm start).
  int64_t idx = -1;
  double w0 = 0.0, w1 = 0.0;
  if (is_col) {
    const int64_t j0 = (int64_t)b * kAuxCols;
    const int ch = threadIdx.x % NCH, grp = threadIdx.x / NCH;
    const int n_rg = a.g.n_rg;
    const int r0 = (int)((int64_t)n_rg * grp / G), r1 = (int)((int64_t)n_rg * (grp + 1) / G);
    const P* cp = static_cast<const P*>(a.colpart) + j0 + ch * CW;
    double s[CW];
#pragma unroll
    for (int e = 0; e < CW; ++e) s[e] = 0.0;
    sum_strided<8>(reinterpret_cast<const V*>(cp), a.g.ldcp / CW, r0, r1, s);
#pragma unroll
    for (int e = 0; e < CW; ++e) red2[grp * kAuxCols + ch * CW + e] = s[e];
    const int64_t j = j0 + threadIdx.x;
    if (threadIdx.x < kAuxCols && j < n) {
      idx = j;
      w0 = (double)static_cast<const T*>(a.q)[j];
      if (is_iter(MODE)) w1 = a.b[j];
      else if (is_final(MODE)) w1 = a.psi64[j];
      else w1 = a.nu0 ? a.nu0[j] : 0.0;
    }
  } else {
    const int64_t i = (int64_t)(b - col_wgs) * kAuxRows + lane;
    double u[1] = {0.0};
    if (i < m) {
      const int n_rp = is_iter(MODE) ? a.g.n_rp : a.g.n_ct;
      const int c0 = n_rp * wave / kWaves, c1 = n_rp * (wave + 1) / kWaves;
      typedef P P1 __attribute__((ext_vector_type(1)));
      sum_strided<8>(reinterpret_cast<const P1*>(static_cast<const P*>(a.rowpart) + i), m, c0, c1,
                     u);
      if (wave == 0) {
        idx = i;
        w0 = (double)static_cast<const T*>(a.p)[i];
        if (is_iter(MODE)) w1 = a.a[i];
        else if (is_final(MODE)) w1 = a.phi64[i];
        else w1 = a.mu0 ? a.mu0[i] : 0.0;
      }
    }
    red2[wave * kAuxRows + lane] = u[0];
  }
  double acc[kSlots];
#pragma unroll
  for (int s = 0; s < kSlots; ++s) acc[s] = 0.0;
  if (wave == 0) {
    // A fixed slice of the sweep's tile scalars, 4 tiles per lane in flight.
    const int64_t nt = (int64_t)a.g.n_ct * a.g.n_rg;
    const int64_t t0 = nt * b / nb, t1 = nt * (b + 1) / nb;
    for (int64_t tb = t0; tb < t1; tb += 4 * kWave) {
      double v0[4], v1[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t t = tb + u * kWave + lane;
        v0[u] = t < t1 ? a.tiles[t * kTileSlots + kTs0] : 0.0;
        v1[u] = t < t1 ? a.tiles[t * kTileSlots + kTs1] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        acc[kST0] += v0[u];
        acc[kST1] += v1[u];
      }
    }
  }
  __syncthreads();
  if (wave != 0 || (is_iter(MODE) && sv.done)) return;

  // Stage 2 (wave 0): the per-entry steps, written once for both kinds of
  // workgroup: `tot` is the entry's full sum (u_i or v_j), `len` the length
  // of the other side (n for rows, m for columns).  The three pointers are
  // picked as values (made wave-uniform first), so that no field of the
  // arguments is ever addressed through a runtime choice.
  const double rho = sv.rho;
  double* const accv = pick(is_col, a.b, a.a);      // a_i or b_j
  double* const d64 = pick(is_col, a.psi64, a.phi64);
  T* const dT = static_cast<T*>(pick(is_col, a.psiT, a.phiT));
  double* const dout = pick(is_col, a.nu_out, a.mu_out);
  const double len = is_col ? (double)m : (double)n;
  const double shift = is_col ? sv.cpsi : sv.cphi;
  const double sum0 = is_col ? sv.sum_phi0 : sv.sum_psi0;
  // e0, e1, e2: the entry's (residual or a_0 / b_0, its square, marginal x dual)
  double e0 = 0.0, e1 = 0.0, e2 = 0.0, emarg = 0.0, esq = 0.0, eneg = 0.0, ebad = 0.0;
  if (idx >= 0) {
    double tot;
    if (is_col) {
      tot = red2[threadIdx.x];
#pragma unroll
      for (int g = 1; g < G; ++g) tot += red2[g * kAuxCols + threadIdx.x];
    } else {
      tot = red2[lane];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) tot += red2[w * kAuxRows + lane];
    }
    const double marg = w0;
    const double res = tot - marg;
    if (is_iter(MODE)) {
      const double d = (w1 - 2.0 * res) / len;
      accv[idx] = w1 - res;
      d64[idx] = d;
      dT[idx] = (T)d;
      e0 = res;
      e1 = res * res;
      e2 = marg * d;
    } else if (is_final(MODE)) {
      const double d = w1 + shift;
      e1 = res * res;
      e2 = marg * d;
      if (dout) dout[idx] = d / rho;
    } else {
      const double d0 = rho * w1;
      const double acc0 = res + len * d0 + sum0;
      accv[idx] = acc0;
      d64[idx] = d0;
      dT[idx] = (T)d0;
      e0 = acc0;
      emarg = marg;
      esq = marg * marg;
      eneg = marg < 0.0 ? 1.0 : 0.0;
      ebad = (!finite_d(marg) || !finite_d(d0)) ? 1.0 : 0.0;
    }
  }

  // Publish this workgroup's sums (slot-major), then count it in; the
  // release fence orders the stores before the count and the acquire fence
  // of the last workgroup orders its loads after it.  Column workgroups fill
  // the column slots, row workgroups the row slots; in the iteration no
  // other slot is read.
  double* const bp = a.blockpart + b;
  const int64_t sb = is_col ? kSS : kSR;  // first of the side's three slots
  unsigned prev = 0;
  if (is_iter(MODE)) {
    double w[5] = {e0, e1, e2, acc[kST0], acc[kST1]};
    wave_sum_n(w);
    if (lane == 0) {
      store_agent(bp + (sb + 0) * nb, w[0]);
      store_agent(bp + (sb + 1) * nb, w[1]);
      store_agent(bp + (sb + 2) * nb, w[2]);
      store_agent(bp + (int64_t)kST0 * nb, w[3]);
      store_agent(bp + (int64_t)kST1 * nb, w[4]);
    }
  } else {
    // Initialisation / final evaluation: all 13 slots, zeros included.
    double w[10] = {e0, e1, e2, emarg, esq, eneg, ebad, acc[kST0], acc[kST1], 0.0};
    wave_sum_n(w);
    const double r0 = is_col ? 0.0 : w[0], r1 = is_col ? 0.0 : w[1], r2 = is_col ? 0.0 : w[2];
    const double c0 = is_col ? w[0] : 0.0, c1 = is_col ? w[1] : 0.0, c2 = is_col ? w[2] : 0.0;
    const double sp = is_col ? 0.0 : w[3], sq = is_col ? w[3] : 0.0;
    if (lane == 0) {
      store_agent(bp + (int64_t)kSR * nb, r0);
      store_agent(bp + (int64_t)kSR2 * nb, r1);
      store_agent(bp + (int64_t)kSPphi * nb, r2);
      store_agent(bp + (int64_t)kSS * nb, c0);
      store_agent(bp + (int64_t)kSS2 * nb, c1);
      store_agent(bp + (int64_t)kSQpsi * nb, c2);
      store_agent(bp + (int64_t)kST0 * nb, w[7]);
      store_agent(bp + (int64_t)kST1 * nb, w[8]);
      store_agent(bp + (int64_t)kSP * nb, sp);
      store_agent(bp + (int64_t)kSQ * nb, sq);
      store_agent(bp + (int64_t)kSPQ2 * nb, w[4]);
      store_agent(bp + (int64_t)kSNeg * nb, w[5]);
      store_agent(bp + (int64_t)kSNonfin * nb, w[6]);
    }
  }
  // Split form: the scalar steps run in a separate one-workgroup launch, and
  // the kernel boundary publishes the sums (no fence per workgroup).
  if constexpr (SPLIT) return;
  if (lane == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    prev = __hip_atomic_fetch_add(&a.st->counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  prev = __builtin_amdgcn_readfirstlane(prev);
  if (prev != (unsigned)(nb - 1)) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  finish_global<MODE>(a, sv, nb, col_wgs, a.st, a.blockpart, a.st);
  if (lane == 0)
    __hip_atomic_store(&a.st->counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T, int MODE, bool WIDE = false, bool SPLIT = false>
__global__ __launch_bounds__(kBlock) void aux_kernel(SweepArgs a) {
  aux_body<T, MODE, WIDE, SPLIT>(a, blockIdx.x, gridDim.x);
}

// The scalar steps after a publish-only aux launch: one wave.  They read the
// record and sums of the aux launch (a.st, a.blockpart), or in the pending
// form (a.st_prev, a.bp_prev), and commit into a.st.
template <int MODE>
__device__ __forceinline__ void finish_body(const SweepArgs& a) {
  const DevState* src = a.st_prev ? a.st_prev : a.st;
  const double* bp = a.st_prev ? a.bp_prev : a.blockpart;
  const StateIn sv = load_state(src);
  if (is_iter(MODE) && sv.done) {
    if (src != a.st && threadIdx.x == 0) *a.st = *src;  // carry the stopped state forward
    return;
  }
  const int nb = (int)aux_workgroups(a.g.m, a.g.n);
  const int col_wgs = (int)((a.g.n + kAuxCols - 1) / kAuxCols);
  finish_global<MODE>(a, sv, nb, col_wgs, src, bp, a.st);
}

template <int MODE>
__global__ __launch_bounds__(kWave) void finish_kernel(SweepArgs a) {
  finish_body<MODE>(a);
}

// Batched form: one wave per problem (finished problems return at once).
template <int MODE>
__global__ __launch_bounds__(kWave) void finish_batch_kernel(const SweepArgs* __restrict__ args) {
  const SweepArgs a = args[blockIdx.x];
  finish_body<MODE>(a);
}

// Batched form: work item = (problem, aux workgroup of that problem).
template <typename T, int MODE>
__global__ __launch_bounds__(kBlock) void aux_batch_kernel(const SweepArgs* __restrict__ args,
                                                           const uint2* __restrict__ work) {
  const uint2 w = work[blockIdx.x];
  // A private copy of the problem's arguments: read through the pointer,
  // every field would be reloaded after each store the kernel makes.
  const SweepArgs a = args[__builtin_amdgcn_readfirstlane(w.x)];
  aux_body<T, MODE, false, true>(a, (int)w.y, (int)aux_workgroups(a.g.m, a.g.n));
}

// The batched iteration's aux work items, one per wave, four per workgroup
// (the batch's items are small: a few row groups deep, so a whole workgroup
// per item spent most of its life on fixed costs).  Per item the same
// quantities as aux_body<T, kIter, false, true> with these orders: column
// items split the row groups over G1 lane groups (each adds its range in
// order) and add the G1 sums in order; row items add their strips in order;
// every lane then takes the step of its column or row.
template <typename T>
__device__ __forceinline__ void aux_wave_iter(const SweepArgs& a, const int b, const int nb,
                                              double* __restrict__ red) {
  using P = typename PartialOf<T, kIter>::type;
  constexpr int CW = 16 / sizeof(P);   // columns per 16-byte chunk
  constexpr int NCH = kAuxCols / CW;   // chunks per item
  constexpr int G1 = kWave / NCH;      // row-group ranges per item (= CW)
  using V = typename VecOf<P, CW>::type;
  static_assert(kAuxCols == kWave && kAuxRows == kWave, "one entry per lane");

  const StateIn sv = load_state(a.st);
  const int64_t m = a.g.m, n = a.g.n;
  const int col_wgs = (int)((n + kAuxCols - 1) / kAuxCols);
  const int lane = threadIdx.x & (kWave - 1);
  const bool is_col = b < col_wgs;

  int64_t idx = -1;
  double w0 = 0.0, w1 = 0.0, tot = 0.0;
  if (is_col) {
    const int64_t j0 = (int64_t)b * kAuxCols;
    const int ch = lane % NCH, grp = lane / NCH;
    const int n_rg = a.g.n_rg;
    const int r0 = (int)((int64_t)n_rg * grp / G1), r1 = (int)((int64_t)n_rg * (grp + 1) / G1);
    const P* cp = static_cast<const P*>(a.colpart) + j0 + ch * CW;
    double sv4[CW];
#pragma unroll
    for (int e = 0; e < CW; ++e) sv4[e] = 0.0;
    sum_strided<8>(reinterpret_cast<const V*>(cp), a.g.ldcp / CW, r0, r1, sv4);
#pragma unroll
    for (int e = 0; e < CW; ++e) red[grp * kAuxCols + ch * CW + e] = sv4[e];
    const int64_t j = j0 + lane;
    if (j < n) {
      idx = j;
      w0 = (double)static_cast<const T*>(a.q)[j];
      w1 = a.b[j];
    }
  } else {
    const int64_t i = (int64_t)(b - col_wgs) * kAuxRows + lane;
    if (i < m) {
      typedef P P1 __attribute__((ext_vector_type(1)));
      double u[1] = {0.0};
      sum_strided<8>(reinterpret_cast<const P1*>(static_cast<const P*>(a.rowpart) + i), m, 0,
                     a.g.n_rp, u);
      tot = u[0];
      idx = i;
      w0 = (double)static_cast<const T*>(a.p)[i];
      w1 = a.a[i];
    }
  }
  // A fixed slice of the sweep's tile scalars.
  double st0 = 0.0, st1 = 0.0;
  {
    const int64_t nt = (int64_t)a.g.n_ct * a.g.n_rg;
    const int64_t t0 = nt * b / nb, t1 = nt * (b + 1) / nb;
    for (int64_t tb = t0; tb < t1; tb += 4 * kWave) {
      double v0[4], v1[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t t = tb + u * kWave + lane;
        v0[u] = t < t1 ? a.tiles[t * kTileSlots + kTs0] : 0.0;
        v1[u] = t < t1 ? a.tiles[t * kTileSlots + kTs1] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        st0 += v0[u];
        st1 += v1[u];
      }
    }
  }
  if (sv.done) return;
  // The column sums cross lanes of this wave through LDS.
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (is_col && idx >= 0) {
    tot = red[lane];
#pragma unroll
    for (int g = 1; g < G1; ++g) tot += red[g * kAuxCols + lane];
  }
  double* const accv = pick(is_col, a.b, a.a);      // a_i or b_j
  double* const d64 = pick(is_col, a.psi64, a.phi64);
  T* const dT = static_cast<T*>(pick(is_col, a.psiT, a.phiT));
  const double len = is_col ? (double)m : (double)n;
  double e0 = 0.0, e1 = 0.0, e2 = 0.0;
  if (idx >= 0) {
    const double res = tot - w0;
    const double d = (w1 - 2.0 * res) / len;
    accv[idx] = w1 - res;
    d64[idx] = d;
    dT[idx] = (T)d;
    e0 = res;
    e1 = res * res;
    e2 = w0 * d;
  }
  double w[5] = {e0, e1, e2, st0, st1};
  wave_sum_n(w);
  if (lane == 0) {
    double* const bp = a.blockpart + b;
    const int64_t sb = is_col ? kSS : kSR;
    store_agent(bp + (sb + 0) * nb, w[0]);
    store_agent(bp + (sb + 1) * nb, w[1]);
    store_agent(bp + (sb + 2) * nb, w[2]);
    store_agent(bp + (int64_t)kST0 * nb, w[3]);
    store_agent(bp + (int64_t)kST1 * nb, w[4]);
  }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void aux_batch_iter_kernel(const SweepArgs* __restrict__ args,
                                                                const uint2* __restrict__ work,
                                                                int64_t n_aux) {
  constexpr int CW = 16 / sizeof(typename PartialOf<T, kIter>::type);
  __shared__ double red[kWaves][CW * kAuxCols];  // per wave: CW row-group ranges x 64 columns
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t item = (int64_t)blockIdx.x * kWaves + wave;
  if (item >= n_aux) return;
  const uint2 w = work[item];
  const SweepArgs a = args[__builtin_amdgcn_readfirstlane(w.x)];  // private copy, as above
  aux_wave_iter<T>(a, (int)__builtin_amdgcn_readfirstlane(w.y), (int)aux_workgroups(a.g.m, a.g.n),
                   red[wave]);
}

// Per-lane accumulator of the sweep.  Plain: a running sum in the partial
// type.  Compensated (float32 iteration with DROT_FLAG_COMPENSATED): a
// Neumaier (improved Kahan-Babuska) pair of floats, so that a lane's sum over
// its entries carries an error of about one rounding whatever its length; the
// pair is handed on as s + c in float64, and every later combination
// (across lanes, waves, tiles) is a float64 sum.
template <typename P, bool KC>
struct LaneAcc {
  P v = 0;
  template <typename X>
  __device__ __forceinline__ void add(X x) { v += (P)x; }
  __device__ __forceinline__ P get() const { return v; }
};

template <>
struct LaneAcc<double, true> {
  float s = 0.f, c = 0.f;
  __device__ __forceinline__ void add(float x) {
    const float t = s + x;
    c += __builtin_fabsf(s) >= __builtin_fabsf(x) ? (s - t) + x : (x - t) + s;
    s = t;
  }
  __device__ __forceinline__ double get() const { return (double)s + (double)c; }
};

// ---------------------------------------------------------------------------
// The sweep.  A workgroup owns one column strip of W = 64 * VEC * CH columns
// and the row blocks g, g + G, g + 2G, ... of `rows` rows each (G = n_rg row
// groups): the workgroups running at any moment stream one contiguous band
// of row blocks (short blocks keep DRAM pages open), while column partials
// are kept per group, so there are G rows of them instead of one per block.
// Within a block the four waves take contiguous slices of rows; each lane
// owns CH chunks of VEC consecutive columns and keeps the loads of U rows in
// flight.  Consecutive workgroups take consecutive strips of the same group.
// ---------------------------------------------------------------------------
template <typename T, int MODE, int VEC, int CH, int U, bool NT, int CM, int D, bool RAGGED,
          bool KC = false>
__device__ __forceinline__ void sweep_body(const SweepArgs& a, const int ct, const int rg) {
  static_assert(!KC || (std::is_same<T, float>::value && MODE == kIter),
                "compensated sums: float32 plain iteration only");
  using P = typename std::conditional<KC, double, typename PartialOf<T, MODE>::type>::type;
  using L = LaneAcc<P, KC>;
  using A = typename std::conditional<is_final(MODE), double, T>::type;
  constexpr int CPL = VEC * CH;
  constexpr int W = kWave * CPL;
  constexpr bool kReadC = MODE != kIterB && CM != kCostCoords;
  static_assert(CM == kCostDense || std::is_same<T, float>::value, "cost kind needs float32");
  constexpr bool kReadX = MODE != kInitPQ;
  constexpr bool kWriteX = MODE != kInitX && MODE != kFinal;

  // The state entering this iteration.  Pending form (a.st_prev set): every
  // wave closes the previous iteration itself from its record and its aux
  // sums (the same fixed-order arithmetic everywhere, so every workgroup
  // takes the same shift and the same stop decision), and workgroup 0
  // commits the result to a.st, which no other workgroup reads here.
  const int64_t m = a.g.m, n = a.g.n;
  const DevState* st = is_iter(MODE) && a.st_prev ? a.st_prev : a.st;
  double shift_d = 0.0;
  if (is_iter(MODE)) {
    if (a.st_prev) {
      // Wave 0 closes the previous iteration and hands the shift and the
      // stop decision to the other waves through LDS.
      __shared__ double closing[2];
      if (threadIdx.x < kWave) {
        // The record's loads first, so that they are in flight with the sums'.
        const StateIn pv = load_state(a.st_prev);
        double w[8];
        iter_sums<false>(a.bp_prev, (int)aux_workgroups(m, n),
                         (int)((n + kAuxCols - 1) / kAuxCols), w);
        double sh = 0.0, stop = 1.0;
        if (pv.done) {
          if (blockIdx.x == 0 && threadIdx.x == 0) *a.st = *a.st_prev;
        } else {
          const ScalarStep f = scalar_step(pv, w, m, n, a.prev_b != 0);
          if (blockIdx.x == 0 && threadIdx.x == 0) commit_step(a.st, a.st_prev, f, a, pv.t_start);
          sh = f.cphi + f.cpsi;
          stop = f.done ? 1.0 : 0.0;
        }
        if (threadIdx.x == 0) {
          closing[0] = sh;
          closing[1] = stop;
        }
      }
      __syncthreads();
      if (closing[1] != 0.0) return;
      shift_d = closing[0];
    } else {
      if (st->done) return;
      shift_d = st->cphi + st->cpsi;
    }
  } else if (is_final(MODE)) {
    shift_d = st->cphi + st->cpsi;
  }

  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t col0 = (int64_t)ct * W;
  const int rpw = (a.g.rows + kWaves - 1) / kWaves;

  const T* __restrict__ C = static_cast<const T*>(a.C);
  const uint16_t* __restrict__ Cb = static_cast<const uint16_t*>(a.C);
  T* __restrict__ X = static_cast<T*>(a.X);

  // Column layout of this lane: chunk c covers [jc[c], jc[c] + VEC), of which
  // nv[c] columns lie inside the matrix.  A chunk that straddles column n is
  // loaded whole (the leading dimensions are multiples of VEC, so the load
  // stays inside the row) but only its valid elements count and are stored.
  int64_t jc[CH];
  int nv[CH];
  bool ok[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    jc[c] = col0 + (int64_t)c * kWave * VEC + (int64_t)lane * VEC;
    const int64_t left = n - jc[c];
    if constexpr (RAGGED) nv[c] = left <= 0 ? 0 : (left >= VEC ? VEC : (int)left);
    else nv[c] = left > 0 ? VEC : 0;  // n is a multiple of VEC
    ok[c] = nv[c] > 0;
  }

  // Column shift of this lane's columns (or q_j for X_0 = p q^T).
  A colv[CH][VEC];
#pragma unroll
  for (int c = 0; c < CH; ++c)
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      A v = 0;
      if (e < nv[c]) {
        const int64_t j = jc[c] + e;
        if (is_iter(MODE)) v = static_cast<const T*>(a.psiT)[j];
        if (is_final(MODE)) v = a.psi64[j];
        if (MODE == kInitPQ) v = static_cast<const T*>(a.q)[j];
      }
      colv[c][e] = v;
    }

  // Coordinates of this lane's target points (coordinates cost only).
  constexpr int DD = CM == kCostCoords ? D : 1;
  float xtl[CH][VEC][DD];
  float cscale = 0.f;
  if constexpr (CM == kCostCoords) {
    cscale = (float)st->cscale;
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int e = 0; e < VEC; ++e)
#pragma unroll
        for (int d = 0; d < D; ++d) xtl[c][e][d] = e < nv[c] ? a.xt[(jc[c] + e) * D + d] : 0.f;
  }

  A shift = 0, rho = 0;
  T rhoT = 0;
  if (is_iter(MODE) || is_final(MODE)) {
    shift = (A)shift_d;
    rho = (A)st->rho;
    rhoT = (T)st->rho;
  }

  L colacc[CH][VEC];
  L s0, s1;  // tile scalars (cost & dual, or |C|^2 & bad count)

  // Where a workgroup takes more than one row block and strips of two chunks by
  // default (kWiden: streamed problems, and costs that are not dense), a lane's
  // plain float32 sums run over U rows and are then added in float64, the
  // columns' in LDS, where they take no registers; and a row has a partial for
  // each chunk (kTwoSums, row_partials()).  So no float32 sum is longer than in
  // strips of one chunk and two row blocks of 16: after an iteration of random
  // plans the row sums' error is that of such strips and the column sums' 0.6 to
  // 0.8 of it, with longer float32 sums 1.4 and 1.5 times (us per iteration with
  // them -> so: 20000 x 20000 768 -> 770, 6000 x 6000 70.0 -> 72.1, coordinates
  // 10000 x 15000 189.4 -> 192.6).
  constexpr bool kWiden = std::is_same<P, float>::value && VEC > 1 && (NT || CM != kCostDense);
  constexpr bool kTwoSums = kWiden && NT && CH == 2;
  using S = typename std::conditional<kWiden, double, P>::type;
  __shared__ __align__(16) S sm[kWaves * W];
  double s0d = 0.0, s1d = 0.0;
  // Where chunk c's column e of lane l lies in a wave's part of sm: widened, two
  // columns side by side in 16 bytes and the lanes next to each other.
  auto slot = [](int c, int e, int l) {
    return kWiden ? ((c * VEC + e) / 2 * kWave + l) * 2 + e % 2 : (c * kWave + l) * VEC + e;
  };
  if constexpr (kWiden) {
#pragma unroll
    for (int k = 0; k < CPL; ++k) sm[wave * W + slot(k / VEC, k % VEC, lane)] = (S)0;
  }

  P* __restrict__ rowpart = static_cast<P*>(a.rowpart);

  // One row block; the policy says whether its accesses are nontemporal.
  auto block = [&](int64_t rb, auto policy) {
    constexpr bool STREAM = decltype(policy)::value;
    const int64_t row0 = rb * a.g.rows;
    const int64_t rowE = row0 + a.g.rows < m ? row0 + a.g.rows : m;
    const int64_t rw0 = row0 + (int64_t)wave * rpw;
    const int64_t rw1 = rw0 + rpw < rowE ? rw0 + rpw : rowE;
    for (int64_t i0 = rw0; i0 < rw1; i0 += U) {
      T xv[U][CH][VEC], cv[U][CH][VEC];
      float xsr[U][DD];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t i = i0 + u;
        if (i < rw1) {
          if constexpr (CM == kCostCoords)
#pragma unroll
            for (int d = 0; d < D; ++d) xsr[u][d] = a.xs[i * D + d];
#pragma unroll
          for (int c = 0; c < CH; ++c) {
            if (ok[c]) {
              if constexpr (kReadC && CM == kCostDense)
                load_chunk<T, VEC, STREAM>(C + i * a.g.ldc + jc[c], cv[u][c]);
              if constexpr (kReadC && CM == kCostBF16)
                load_bf16<VEC, STREAM>(Cb + i * a.g.ldc + jc[c], cv[u][c]);
              if (kReadX) load_chunk<T, VEC, STREAM>(X + i * a.g.ldx + jc[c], xv[u][c]);
            }
          }
        }
      }
      // c_ij as the storage type sees it.
      auto cost = [&](int u, int c, int e) -> T {
        if constexpr (CM == kCostCoords) {
          float s = 0.f;
#pragma unroll
          for (int d = 0; d < D; ++d) {
            const float df = xsr[u][d] - xtl[c][e][d];
            s += df * df;
          }
          return (T)(s * cscale);
        } else {
          return cv[u][c][e];
        }
      };
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t i = i0 + u;
        if (i < rw1) {
          A rowv = 0;
          if (is_iter(MODE)) rowv = static_cast<const T*>(a.phiT)[i] + shift;
          if (is_final(MODE)) rowv = a.phi64[i] + (double)shift;
          if (MODE == kInitPQ) rowv = static_cast<const T*>(a.p)[i];
          L rsum, rsum0;
#pragma unroll
          for (int c = 0; c < CH; ++c) {
            if (kTwoSums && c == 1) {
              rsum0 = rsum;
              rsum = L{};
            }
            if (ok[c]) {
              T outv[VEC];
#pragma unroll
              for (int e = 0; e < VEC; ++e) {
                A x = 0;
                if (RAGGED && e >= nv[c]) {
                  // beyond column n (padding): contributes nothing, never stored
                  outv[e] = (T)0;
                } else if constexpr (MODE == kIterB) {
                  // X_{k+2} = [W + phi_i + psi_j]_+ with W = X_{k+1} - rho C.
                  const A y = (A)xv[u][c][e] + (rowv + colv[c][e]);
                  x = y > (A)0 ? y : (A)0;
                  outv[e] = (T)x;
                } else if constexpr (is_iter(MODE) || is_final(MODE)) {
                  const A cij = (A)cost(u, c, e);
                  const A pc = is_final(MODE) ? rho * cij : mul_rounded<A>(rho, cij);
                  const A t = rowv + colv[c][e] - pc;
                  const A tp = t > (A)0 ? t : (A)0;
                  s1.add(tp * tp);
                  if constexpr (MODE == kFinalW) {
                    // Restore X from W in the stored type, with the product the
                    // C-reading iteration subtracted.
                    const T pcT = mul_rounded<T>(rhoT, cv[u][c][e]);
                    const T xr = xv[u][c][e] + pcT;
                    outv[e] = xr;
                    x = (A)xr;
                  } else if constexpr (MODE == kFinal) {
                    x = (A)xv[u][c][e];
                  } else {
                    const A y = (A)xv[u][c][e] + t;
                    x = y > (A)0 ? y : (A)0;
                    outv[e] = MODE == kIterA ? (T)(x - pc) : (T)x;
                  }
                  s0.add(cij * x);
                } else {
                  const A cij = (A)cost(u, c, e);
                  if (MODE == kInitPQ) x = rowv * colv[c][e];
                  else x = (A)xv[u][c][e];
                  s0.add((double)cij * (double)cij);
                  const bool bad = !finite_d((double)cij) || !finite_d((double)x) ||
                                   (MODE == kInitX && x < (A)0);
                  s1.add(bad ? (P)1 : (P)0);
                  outv[e] = (T)x;
                }
                rsum.add(x);
                colacc[c][e].add(x);
              }
              if (kWriteX) {
                if (!RAGGED || nv[c] == VEC) {
                  store_chunk<T, VEC, STREAM>(X + i * a.g.ldx + jc[c], outv);
                } else {
#pragma unroll
                  for (int e = 0; e < VEC; ++e)
                    if (e < nv[c]) X[i * a.g.ldx + jc[c] + e] = outv[e];
                }
              }
            }
          }
          const P tot = wave_sum(rsum.get());
          if constexpr (kTwoSums) {
            const P tot0 = wave_sum(rsum0.get());
            if (lane < 2) rowpart[(2 * (int64_t)ct + lane) * m + i] = lane == 0 ? tot0 : tot;
          } else {
            if (lane == 0) rowpart[(int64_t)ct * m + i] = tot;
          }
        }
      }
      if constexpr (kWiden) {
        // nothing of the next rows in here: it would cost a wave per SIMD
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
          for (int e = 0; e < VEC; ++e) {
            sm[wave * W + slot(c, e, lane)] += (S)colacc[c][e].get();
            colacc[c][e] = L{};
          }
        s0d += (double)s0.get();
        s1d += (double)s1.get();
        s0 = s1 = L{};
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  for (int64_t rb = rg; rb < a.g.n_rb; rb += a.g.n_rg) {
    if constexpr (NT && !KC) {
      // keep of every 1024 row blocks, evenly spread: each time the running
      // multiple of keep passes a multiple of 1024.
      if ((int)((uint32_t)rb * (uint32_t)a.g.keep & 1023u) < a.g.keep)
        block(rb, std::integral_constant<bool, false>{});
      else
        block(rb, std::integral_constant<bool, true>{});
    } else {
      block(rb, std::integral_constant<bool, NT>{});
    }
  }

  // ---- tile partials: combine the four waves in LDS, fixed order -----------
  __shared__ double ssc[2][kWaves];
  if constexpr (kWiden) {
    s0d = wave_sum(s0d);
    s1d = wave_sum(s1d);
  } else {
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int e = 0; e < VEC; ++e) sm[wave * W + slot(c, e, lane)] = colacc[c][e].get();
    s0d = (double)wave_sum(s0.get());
    s1d = (double)wave_sum(s1.get());
  }
  if (lane == 0) {
    ssc[0][wave] = s0d;
    ssc[1][wave] = s1d;
  }
  __syncthreads();
  P* __restrict__ colpart = static_cast<P*>(a.colpart);
  for (int k = threadIdx.x; k < W; k += kBlock) {
    const int64_t j = col0 + k;
    if (j < n) {
      const int at = slot(k / (kWave * VEC), k % VEC, k / VEC % kWave);
      S v = sm[at];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) v += sm[w * W + at];
      colpart[(int64_t)rg * a.g.ldcp + j] = (P)v;
    }
  }
  if (threadIdx.x == 0) {
    double v0 = ssc[0][0], v1 = ssc[1][0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
      v0 += ssc[0][w];
      v1 += ssc[1][w];
    }
    double* t = a.tiles + ((int64_t)rg * a.g.n_ct + ct) * kTileSlots;
    t[kTs0] = v0;
    t[kTs1] = v1;
  }
}

template <typename T, int MODE, int VEC, int CH, int U, bool NT, int CM, int D, bool RAGGED,
          bool KC>
__global__ __launch_bounds__(kBlock) void sweep_kernel(SweepArgs a) {
  sweep_body<T, MODE, VEC, CH, U, NT, CM, D, RAGGED, KC>(a, blockIdx.x % a.g.n_ct,
                                                          blockIdx.x / a.g.n_ct);
}

// Batched form: work item = (problem, workgroup of that problem's sweep).
template <typename T, int MODE, int VEC, int CH, bool NT, bool RAGGED>
__global__ __launch_bounds__(kBlock) void sweep_batch_kernel(const SweepArgs* __restrict__ args,
                                                             const uint2* __restrict__ work) {
  const uint2 w = work[blockIdx.x];
  const SweepArgs a = args[__builtin_amdgcn_readfirstlane(w.x)];  // private copy, as above
  sweep_body<T, MODE, VEC, CH, 4, NT, kCostDense, 1, RAGGED>(a, (int)(w.y % a.g.n_ct),
                                                              (int)(w.y / a.g.n_ct));
}

// Warm-start sums sum(phi_0) = rho sum(mu0), sum(psi_0) = rho sum(nu0), the
// start timestamp, and zeroed completion counters.  One workgroup.
__device__ __forceinline__ void prep_body(const SweepArgs& a) {
  __shared__ double red[kSlots][kWaves];
  double acc[kSlots];
#pragma unroll
  for (int s = 0; s < kSlots; ++s) acc[s] = 0.0;
  if (a.mu0)
    for (int64_t i = threadIdx.x; i < a.g.m; i += kBlock) acc[0] += a.mu0[i];
  if (a.nu0)
    for (int64_t j = threadIdx.x; j < a.g.n; j += kBlock) acc[1] += a.nu0[j];
  block_sum_slots(acc, red);
  if (threadIdx.x == 0) {
    DevState* st = a.st;
    st->sum_phi0 = st->rho * acc[0];
    st->sum_psi0 = st->rho * acc[1];
    if (a.cost_kind == kCostCoords && !(st->cscale > 0.0)) {
      const float mx = __uint_as_float(st->maxc_bits);
      st->cscale = mx > 0.f ? 1.0 / (double)mx : 1.0;
    }
    st->t_start = wall_clock64();
    st->t_stop = st->t_start;
    st->t_last = st->t_start;
    st->counter = 0;
  }
}

__global__ __launch_bounds__(kBlock) void prep_kernel(SweepArgs a) { prep_body(a); }

__global__ __launch_bounds__(kBlock) void prep_batch_kernel(const SweepArgs* __restrict__ args) {
  const SweepArgs a = args[blockIdx.x];
  prep_body(a);
}

// Stream of a sweep launch, with optional events that hipExtLaunchKernel
// stamps with the dispatch's own start and end times.
struct Launch {
  hipStream_t s;
  hipEvent_t e0, e1;
};

template <typename T, int MODE, int VEC, int CH, int U, bool NT, int CM = kCostDense, int D = 1,
          bool RAGGED = false, bool KC = false>
hipError_t sweep_go(const SweepArgs& a, const Launch& s) {
  const dim3 grid((unsigned)((int64_t)a.g.n_ct * a.g.n_rg));
  if (s.e0 || s.e1)
    hipExtLaunchKernelGGL((sweep_kernel<T, MODE, VEC, CH, U, NT, CM, D, RAGGED, KC>), grid,
                          dim3(kBlock), 0, s.s, s.e0, s.e1, 0, a);
  else
    hipLaunchKernelGGL((sweep_kernel<T, MODE, VEC, CH, U, NT, CM, D, RAGGED, KC>), grid,
                       dim3(kBlock), 0, s.s, a);
  return hipGetLastError();
}

// The compensated float32 iteration: 16-byte path with 1 or 2 chunks, 4 rows
// in flight, cached or streaming; the scalar path with 4 chunks (which the
// host also uses for ragged widths).
template <int CM, int D>
hipError_t sweep_comp(const TileCfg& t, const SweepArgs& a, const Launch& s) {
  if (t.ragged || t.unroll != 4) return hipErrorInvalidValue;
  if (t.vec == 1) {
    if (t.chunks != 4) return hipErrorInvalidValue;
    return sweep_go<float, kIter, 1, 4, 4, false, CM, D, false, true>(a, s);
  }
  if (t.vec != 4) return hipErrorInvalidValue;
  switch ((t.chunks == 2 ? 1 : 0) | (t.stream ? 2 : 0)) {
    case 0: return sweep_go<float, kIter, 4, 1, 4, false, CM, D, false, true>(a, s);
    case 1: return sweep_go<float, kIter, 4, 2, 4, false, CM, D, false, true>(a, s);
    case 2: return sweep_go<float, kIter, 4, 1, 4, true, CM, D, false, true>(a, s);
    case 3: return sweep_go<float, kIter, 4, 2, 4, true, CM, D, false, true>(a, s);
  }
  return hipErrorInvalidValue;
}

// 16-byte path with n not a multiple of the vector width (masked last chunk):
// 1 or 2 chunks, 4 rows in flight, cached or streaming.
template <typename T, int MODE, int CM, int D>
hipError_t sweep_ragged(const TileCfg& t, const SweepArgs& a, const Launch& s) {
  constexpr int V = 16 / sizeof(T);
  if (t.vec != V || t.unroll != 4) return hipErrorInvalidValue;
  switch ((t.chunks == 2 ? 1 : 0) | (t.stream ? 2 : 0)) {
    case 0: return sweep_go<T, MODE, V, 1, 4, false, CM, D, true>(a, s);
    case 1: return sweep_go<T, MODE, V, 2, 4, false, CM, D, true>(a, s);
    case 2: return sweep_go<T, MODE, V, 1, 4, true, CM, D, true>(a, s);
    case 3: return sweep_go<T, MODE, V, 2, 4, true, CM, D, true>(a, s);
  }
  return hipErrorInvalidValue;
}

// The iteration instantiates every tile variant; initialisation and the final
// evaluation run once per solve and use the plain 4-row variant.
template <typename T, int MODE>
hipError_t sweep_dense(const TileCfg& t, const SweepArgs& a, const Launch& s) {
  constexpr int V = 16 / sizeof(T);
  if (t.ragged) return sweep_ragged<T, MODE, kCostDense, 1>(t, a, s);
  if (t.vec == 1) {
    if (t.chunks == 1) return sweep_go<T, MODE, 1, 1, 4, false>(a, s);
    if (t.chunks == 4) return sweep_go<T, MODE, 1, 4, 4, false>(a, s);
    return hipErrorInvalidValue;
  }
  if (t.vec != V) return hipErrorInvalidValue;
  if constexpr (is_iter(MODE)) {
    const int key = (t.chunks == 2 ? 1 : 0) | (t.unroll == 8 ? 2 : 0) | (t.stream ? 4 : 0);
    switch (key) {
      case 0: return sweep_go<T, MODE, V, 1, 4, false>(a, s);
      case 1: return sweep_go<T, MODE, V, 2, 4, false>(a, s);
      case 2: return sweep_go<T, MODE, V, 1, 8, false>(a, s);
      case 3: return sweep_go<T, MODE, V, 2, 8, false>(a, s);
      case 4: return sweep_go<T, MODE, V, 1, 4, true>(a, s);
      case 5: return sweep_go<T, MODE, V, 2, 4, true>(a, s);
      case 6: return sweep_go<T, MODE, V, 1, 8, true>(a, s);
      case 7: return sweep_go<T, MODE, V, 2, 8, true>(a, s);
    }
    return hipErrorInvalidValue;
  } else {
    if (t.chunks == 1) return sweep_go<T, MODE, V, 1, 4, false>(a, s);
    if (t.chunks == 2) return sweep_go<T, MODE, V, 2, 4, false>(a, s);
    return hipErrorInvalidValue;
  }
}

// Non-dense cost sources (float32 only): 1 or 2 chunks, 4 rows in flight,
// cached or streaming; the scalar path uses 4 chunks, cached.
template <int MODE, int CM, int D>
hipError_t sweep_cost(const TileCfg& t, const SweepArgs& a, const Launch& s) {
  if (t.ragged) return sweep_ragged<float, MODE, CM, D>(t, a, s);
  if (t.vec == 1) {
    if (t.chunks == 4) return sweep_go<float, MODE, 1, 4, 4, false, CM, D>(a, s);
    return hipErrorInvalidValue;
  }
  if (t.vec != 4 || t.unroll != 4) return hipErrorInvalidValue;
  const int key = (t.chunks == 2 ? 1 : 0) | (t.stream ? 2 : 0);
  switch (key) {
    case 0: return sweep_go<float, MODE, 4, 1, 4, false, CM, D>(a, s);
    case 1: return sweep_go<float, MODE, 4, 2, 4, false, CM, D>(a, s);
    case 2: return sweep_go<float, MODE, 4, 1, 4, true, CM, D>(a, s);
    case 3: return sweep_go<float, MODE, 4, 2, 4, true, CM, D>(a, s);
  }
  return hipErrorInvalidValue;
}

template <typename T, int MODE>
hipError_t sweep_mode(const TileCfg& t, const SweepArgs& a, const Launch& s) {
  if (t.comp) {
    if constexpr (std::is_same<T, float>::value && MODE == kIter) {
      switch (a.cost_kind) {
        case kCostDense: return sweep_comp<kCostDense, 1>(t, a, s);
        case kCostBF16: return sweep_comp<kCostBF16, 1>(t, a, s);
        case kCostCoords:
          if (a.dim == 1) return sweep_comp<kCostCoords, 1>(t, a, s);
          if (a.dim == 2) return sweep_comp<kCostCoords, 2>(t, a, s);
          if (a.dim == 3) return sweep_comp<kCostCoords, 3>(t, a, s);
      }
      return hipErrorInvalidValue;
    }
    // Initialisation and the final evaluation already accumulate in float64.
    if constexpr (MODE == kIter || MODE == kIterA || MODE == kIterB) return hipErrorInvalidValue;
  }
  if (a.cost_kind == kCostDense) return sweep_dense<T, MODE>(t, a, s);
  if constexpr (std::is_same<T, float>::value && !(MODE == kIterA || MODE == kIterB ||
                                                   MODE == kFinalW)) {
    if (a.cost_kind == kCostBF16) return sweep_cost<MODE, kCostBF16, 1>(t, a, s);
    if (a.cost_kind == kCostCoords) {
      switch (a.dim) {
        case 1: return sweep_cost<MODE, kCostCoords, 1>(t, a, s);
        case 2: return sweep_cost<MODE, kCostCoords, 2>(t, a, s);
        case 3: return sweep_cost<MODE, kCostCoords, 3>(t, a, s);
      }
    }
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t sweep_type(int mode, const TileCfg& t, const SweepArgs& a, const Launch& s) {
  switch (mode) {
    case kIter: return sweep_mode<T, kIter>(t, a, s);
    case kInitPQ: return sweep_mode<T, kInitPQ>(t, a, s);
    case kInitX: return sweep_mode<T, kInitX>(t, a, s);
    case kFinal: return sweep_mode<T, kFinal>(t, a, s);
    case kIterA: return sweep_mode<T, kIterA>(t, a, s);
    case kIterB: return sweep_mode<T, kIterB>(t, a, s);
    case kFinalW: return sweep_mode<T, kFinalW>(t, a, s);
  }
  return hipErrorInvalidValue;
}

// max_ij |xs_i - xt_j|^2 for the coordinates cost (scale = 1 / max when the
// caller gives none).  A block covers 256 targets and up to 256 sources; the
// maximum of nonnegative floats is taken on their bit patterns, which order
// the same way, so the result does not depend on the order of the atomics.
template <int D>
__global__ __launch_bounds__(kBlock) void maxc_kernel(SweepArgs a) {
  const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t i0 = (int64_t)blockIdx.y * kBlock;
  const int64_t i1 = i0 + kBlock < a.g.m ? i0 + kBlock : a.g.m;
  float mx = 0.f;
  if (j < a.g.n) {
    float yt[D];
#pragma unroll
    for (int d = 0; d < D; ++d) yt[d] = a.xt[j * D + d];
    for (int64_t i = i0; i < i1; ++i) {
      float s = 0.f;
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const float df = a.xs[i * D + d] - yt[d];
        s += df * df;
      }
      mx = s > mx ? s : mx;
    }
  }
  for (int off = kWave / 2; off > 0; off /= 2) {
    const float o = __shfl_xor(mx, off);
    mx = o > mx ? o : mx;
  }
  if ((threadIdx.x & (kWave - 1)) == 0) atomicMax(&a.st->maxc_bits, __float_as_uint(mx));
}

// One aux launch in the form chosen by the workgroup count: with many
// workgroups the last-arriving election costs one L2 write-back per workgroup
// (its release fence), so above kAuxSplitMin workgroups the aux kernel only
// publishes its sums and a one-wave kernel does the scalar steps.
template <typename T, int MODE, bool WIDE>
hipError_t aux_go(const SweepArgs& a, hipStream_t s, bool publish) {
  const int64_t nb = aux_workgroups(a.g.m, a.g.n);
  const dim3 grid((unsigned)nb);
  if (publish) {
    hipLaunchKernelGGL((aux_kernel<T, MODE, WIDE, true>), grid, dim3(kBlock), 0, s, a);
  } else if (nb >= kAuxSplitMin) {
    hipLaunchKernelGGL((aux_kernel<T, MODE, WIDE, true>), grid, dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL((finish_kernel<MODE>), dim3(1), dim3(kWave), 0, s, a);
  } else {
    hipLaunchKernelGGL((aux_kernel<T, MODE, WIDE, false>), grid, dim3(kBlock), 0, s, a);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t aux_type(int mode, bool wide, const SweepArgs& a, hipStream_t s, bool publish) {
  if (publish && !is_iter(mode)) return hipErrorInvalidValue;
  if (wide && std::is_same<T, float>::value) {
    // Float64 partials of the compensated float32 iteration.
    if (mode != kIter) return hipErrorInvalidValue;
    return aux_go<T, kIter, true>(a, s, publish);
  }
  switch (mode) {
    case kIter:
    case kIterA: return aux_go<T, kIter, false>(a, s, publish);
    case kIterB: return aux_go<T, kIterB, false>(a, s, publish);
    case kInitPQ:
    case kInitX: return aux_go<T, kInitPQ, false>(a, s, false);
    case kFinal:
    case kFinalW: return aux_go<T, kFinal, false>(a, s, false);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_aux(int dtype, int mode, const SweepArgs& a, hipStream_t s, bool wide,
                      bool publish) {
  return dtype == 0 ? aux_type<float>(mode, wide, a, s, publish)
                    : aux_type<double>(mode, wide, a, s, publish);
}

hipError_t launch_finish(int mode, const SweepArgs& a, hipStream_t s) {
  if (mode == kIter || mode == kIterA)
    hipLaunchKernelGGL((finish_kernel<kIter>), dim3(1), dim3(kWave), 0, s, a);
  else if (mode == kIterB)
    hipLaunchKernelGGL((finish_kernel<kIterB>), dim3(1), dim3(kWave), 0, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_sweep(int dtype, int mode, const TileCfg& t, const SweepArgs& a,
                        hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const Launch L{s, e0, e1};
  return dtype == 0 ? sweep_type<float>(mode, t, a, L) : sweep_type<double>(mode, t, a, L);
}

namespace {

template <typename T, int MODE>
hipError_t sweep_batch_mode(const TileCfg& t, const SweepArgs* args, const uint2* work,
                            int64_t nwork, hipStream_t s) {
  constexpr int V = 16 / sizeof(T);
  const dim3 grid((unsigned)nwork), block(kBlock);
  if (t.vec == 1 && t.chunks == 4) {
    hipLaunchKernelGGL((sweep_batch_kernel<T, MODE, 1, 4, false, false>), grid, block, 0, s, args, work);
    return hipGetLastError();
  }
  if (t.vec != V || t.unroll != 4) return hipErrorInvalidValue;
  switch ((t.chunks == 2 ? 1 : 0) | (t.stream ? 2 : 0)) {
    case 0: hipLaunchKernelGGL((sweep_batch_kernel<T, MODE, V, 1, false, true>), grid, block, 0, s, args, work); break;
    case 1: hipLaunchKernelGGL((sweep_batch_kernel<T, MODE, V, 2, false, true>), grid, block, 0, s, args, work); break;
    case 2: hipLaunchKernelGGL((sweep_batch_kernel<T, MODE, V, 1, true, true>), grid, block, 0, s, args, work); break;
    case 3: hipLaunchKernelGGL((sweep_batch_kernel<T, MODE, V, 2, true, true>), grid, block, 0, s, args, work); break;
  }
  return hipGetLastError();
}

// Batched aux: every workgroup publishes its sums, then one wave per problem
// does the scalar steps (a per-workgroup release fence would cost one L2
// write-back per workgroup of every problem).
template <typename T, int MODE>
void batch_aux(const SweepArgs* args, const uint2* aux_work, int64_t n_aux, int n_prob,
               hipStream_t s) {
  if constexpr (MODE == kIter)
    hipLaunchKernelGGL((aux_batch_iter_kernel<T>), dim3((unsigned)((n_aux + kWaves - 1) / kWaves)),
                       dim3(kBlock), 0, s, args, aux_work, n_aux);
  else
    hipLaunchKernelGGL((aux_batch_kernel<T, MODE>), dim3((unsigned)n_aux), dim3(kBlock), 0, s, args,
                       aux_work);
  hipLaunchKernelGGL((finish_batch_kernel<MODE>), dim3((unsigned)n_prob), dim3(kWave), 0, s, args);
}

template <typename T>
hipError_t batch_type(int mode, const TileCfg& t, const SweepArgs* args, const uint2* sweep_work,
                      int64_t n_sweep, const uint2* aux_work, int64_t n_aux, int n_prob,
                      hipStream_t s) {
  hipError_t e = hipSuccess;
  switch (mode) {
    case kIter:
      e = sweep_batch_mode<T, kIter>(t, args, sweep_work, n_sweep, s);
      if (e == hipSuccess) batch_aux<T, kIter>(args, aux_work, n_aux, n_prob, s);
      break;
    case kInitPQ:
    case kInitX:
      e = mode == kInitPQ ? sweep_batch_mode<T, kInitPQ>(t, args, sweep_work, n_sweep, s)
                          : sweep_batch_mode<T, kInitX>(t, args, sweep_work, n_sweep, s);
      if (e == hipSuccess) batch_aux<T, kInitPQ>(args, aux_work, n_aux, n_prob, s);
      break;
    case kFinal:
      e = sweep_batch_mode<T, kFinal>(t, args, sweep_work, n_sweep, s);
      if (e == hipSuccess) batch_aux<T, kFinal>(args, aux_work, n_aux, n_prob, s);
      break;
    default: return hipErrorInvalidValue;
  }
  return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace

hipError_t launch_batch_step(int dtype, int mode, const TileCfg& t, const SweepArgs* args,
                             const uint2* sweep_work, int64_t n_sweep, const uint2* aux_work,
                             int64_t n_aux, int n_prob, hipStream_t s) {
  if (n_sweep <= 0 || n_aux <= 0) return hipSuccess;
  return dtype == 0
             ? batch_type<float>(mode, t, args, sweep_work, n_sweep, aux_work, n_aux, n_prob, s)
             : batch_type<double>(mode, t, args, sweep_work, n_sweep, aux_work, n_aux, n_prob, s);
}

hipError_t launch_prep_batch(const SweepArgs* args, int count, hipStream_t s) {
  hipLaunchKernelGGL(prep_batch_kernel, dim3((unsigned)count), dim3(kBlock), 0, s, args);
  return hipGetLastError();
}

namespace {
template <typename T>
hipError_t small_type(const SweepArgs& a, int64_t iters, hipStream_t s) {
  const dim3 grid(1), block(kSmallBlock);
  switch (small_cols(a.g.n)) {
    case 1: hipLaunchKernelGGL((small_kernel<T, 1>), grid, block, 0, s, a, iters); break;
    case 2: hipLaunchKernelGGL((small_kernel<T, 2>), grid, block, 0, s, a, iters); break;
    case 4: hipLaunchKernelGGL((small_kernel<T, 4>), grid, block, 0, s, a, iters); break;
    case 8: hipLaunchKernelGGL((small_kernel<T, 8>), grid, block, 0, s, a, iters); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
}  // namespace

hipError_t launch_small(int dtype, const SweepArgs& a, int64_t iters, hipStream_t s) {
  // The kernel's register and LDS arrays are sized for small_fits shapes.
  if (!small_fits(dtype, a.g.m, a.g.n)) return hipErrorInvalidValue;
  return dtype == 0 ? small_type<float>(a, iters, s) : small_type<double>(a, iters, s);
}

hipError_t launch_maxc(const SweepArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)((a.g.n + kBlock - 1) / kBlock), (unsigned)((a.g.m + kBlock - 1) / kBlock));
  switch (a.dim) {
    case 1: hipLaunchKernelGGL(maxc_kernel<1>, grid, dim3(kBlock), 0, s, a); break;
    case 2: hipLaunchKernelGGL(maxc_kernel<2>, grid, dim3(kBlock), 0, s, a); break;
    case 3: hipLaunchKernelGGL(maxc_kernel<3>, grid, dim3(kBlock), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_prep(const SweepArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(prep_kernel, dim3(1), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

}  // namespace drot
