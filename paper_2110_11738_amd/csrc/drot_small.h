// Small problems: the whole iteration in one workgroup, thousands of
// iterations per launch, with the plan and rho C in registers.
//
// Eleven sweep waves hold the plan: wave w the rows w, w + 11, ..., lane l the
// columns l, l + 64, ... (NCOL of them).  The twelfth wave, the service wave,
// has the columns' duals and the scalars.  An iteration is
//  - sweep waves: step 4 on their entries.  Each lane's partial of every row
//    goes to LDS as it is, its column sums (float64) too;
//  - barrier;
//  - service wave: column sums over the waves, their total, beta, steps 5-8 of
//    the columns and the scalar parts of the shifts (tall float64 problems: alpha
//    once more at the end, from the rows' residuals).  Meanwhile the sweep
//    waves add their own rows' partials, four lanes per row, and take steps
//    5-8 of the rows;
//  - barrier.
// The stopping test is not in that chain: the service wave takes it while the
// others are in the next sweep, and the next barrier announces a stop.  X has
// moved on by one iteration by then.  So every kSmallSnap iterations, once the
// test of the iteration before is known to have passed, the state goes to
// memory; after a stop the workgroup loads it and repeats the few iterations
// up to the stopping one (everything is deterministic).
//
// Of a float32 problem a lane's sum of a row (at most 8 entries) and its <rho C,X>
// and sum [t]_+^2 of a group of rows (at most 24 entries) are float32, every other
// sum float64.
//
// What bounds it: for the largest shapes the vector units of one compute unit
// (some 12 operations per entry, 64 lanes per clock: 2.6 us of a 256 x 128
// iteration), for the smallest the chain of two barriers, the column sums, the
// sum over the wave and a Newton division each for beta and the shifts, with
// the test (five divisions, two roots) just about fitting beside it.  A test
// inside the chain and the row and column steps one after the other in two
// waves took 4.4 us per iteration at 100 x 100.
// Measured per iteration against that: float32 10 x 10 4.3 -> 1.5 us,
// 100 x 100 4.4 -> 2.05, 256 x 128 5.4 -> 3.2, 512 x 64 6.9 -> 4.1,
// 64 x 512 5.3 -> 3.0; float64 100 x 100 4.6 -> 2.2, 256 x 64 5.1 -> 2.8.
#pragma once

#include "drot_device.h"
#include "drot_internal.h"

namespace drot {
namespace {

// The workgroup's barrier.  The sweep waves and the service wave reach it in
// different places of the program, the same number of times.
__device__ __forceinline__ void small_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Keeps what is made from `v` (addresses, comparisons) from being carried
// through the iterations in registers that the plan needs.
__device__ __forceinline__ int small_fresh(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

template <typename T, int NCOL>
struct SmallShared {
  static constexpr int NW = kSmallWaves;
  static constexpr int RT = small_wave_rows(std::is_same<T, float>::value ? 0 : 1, NCOL);
  T rowp[NW][RT][kWave];         // each lane's partial of each row
  T rowsh[NW][RT];               // row shifts without the scalar part
  double colp[NW][kWave * NCOL];  // column sums of each wave
  double mon0[2][NW][kWave];     // <rho C,X> (lanes < 32), sum [t]_+^2; by parity
  double mon1[NW][kWave];        // sum r^2 (lanes < 32), sum p phi~
  // Float64: sum r, of every fourth lane of the waves; zeros at the end.
  static constexpr int NR = std::is_same<T, double>::value ? (NW + 3) / 4 : 0;
  double rsum[NR ? NR * kWave : 1];
  T colsh[kWave * NCOL];         // column shifts without the scalar part
  T shift;                       // the scalar part, of rows and columns together
  int stop;                      // the iteration of this launch that ended the solve, or 0
};

// Waves 0 .. 10.
template <typename T, int NCOL>
__device__ __forceinline__ void small_sweep(SmallShared<T, NCOL>& sh, const SweepArgs& a,
                                            const T rhoT, int limit) {
  constexpr int NW = kSmallWaves, RT = SmallShared<T, NCOL>::RT;
  constexpr int GR = RT % 4 == 0 ? 4 : 3;  // rows between two looks at the row count
  constexpr int NP = (RT + 15) / 16;       // passes of 16 rows over the wave's row sums
  constexpr int VEC = 16 / sizeof(T), Q = 16 / VEC;  // a quarter row: Q chunks of VEC
  static_assert(RT % GR == 0, "row groups");
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  const int m = (int)a.g.m, n = (int)a.g.n;
  // Rows of this wave: wave + NW t, t < nrows.
  const int nrows = m > wave ? (m - wave + NW - 1) / NW : 0;
  const double dn = (double)n, in = 1.0 / dn;

  T xr[RT][NCOL], pc[RT][NCOL];
  double ra[NP], rph[NP];  // a, phi~ of row 16 p + lane / 4 of the wave
  T marg[NP];

  // rho C once; outside the matrix a cost so large that such entries stay 0.
  {
    const T* C = static_cast<const T*>(a.C) + lane;
    const T kFar = std::is_same<T, float>::value ? (T)3e38f : (T)1e300;
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const T* const row = C + (int64_t)(wave + NW * t) * a.g.ldc;
#pragma unroll
      for (int c = 0; c < NCOL; ++c)
        pc[t][c] = t < nrows && lane + kWave * c < n ? mul_rounded<T>(rhoT, row[kWave * c]) : kFar;
    }
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int r = 16 * p + (lane >> 2);
    marg[p] = r < nrows ? static_cast<const T*>(a.p)[wave + NW * r] : (T)0;
  }

  int base_k = 0, k = 0;
  bool replay = false;
  for (;;) {  // from the state in memory on: the launch, and after a stop once more
    k = base_k;
    {
      int w = small_fresh(wave);
      const int nr = small_fresh(nrows), nn = small_fresh(n);
      const T* X = static_cast<const T*>(a.X) + lane;
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const T* const row = X + (int64_t)(w + NW * t) * a.g.ldx;
#pragma unroll
        for (int c = 0; c < NCOL; ++c)
          xr[t][c] = t < nr && lane + kWave * c < nn ? row[kWave * c] : (T)0;
      }
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const int r = 16 * p + (lane >> 2);
        ra[p] = r < nr ? a.a[w + NW * r] : 0.0;
        rph[p] = r < nr ? a.phi64[w + NW * r] : 0.0;
      }
      for (int r = lane; r < RT; r += kWave)
        sh.rowsh[w][r] = r < nr ? static_cast<const T*>(a.phiT)[w + NW * r] : (T)0;
    }
    small_barrier();

    auto save = [&]() {
      int w = small_fresh(wave);
      const int nr = small_fresh(nrows), nn = small_fresh(n);
      T* X = static_cast<T*>(a.X) + lane;
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        T* const row = X + (int64_t)(w + NW * t) * a.g.ldx;
#pragma unroll
        for (int c = 0; c < NCOL; ++c)
          if (t < nr && lane + kWave * c < nn) row[kWave * c] = xr[t][c];
      }
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const int r = 16 * p + (lane >> 2);
        if ((lane & 3) == 0 && r < nr) {
          a.a[w + NW * r] = ra[p];
          a.phi64[w + NW * r] = rph[p];
          static_cast<T*>(a.phiT)[w + NW * r] = (T)rph[p];
        }
      }
    };

    bool stopped = false;
    while (k < limit) {
      const int nr = small_fresh(nrows);
      // Step 4 on the held entries; <rho C,X> and sum [t]_+^2 at the incoming
      // shifts.
      {
        const T shift = sh.shift;
        T colv[NCOL];
        double cd[NCOL], s0d = 0.0, s1d = 0.0;
#pragma unroll
        for (int c = 0; c < NCOL; ++c) {
          colv[c] = sh.colsh[lane + kWave * c];
          cd[c] = 0.0;
        }
#pragma unroll
        for (int g = 0; g < RT / GR; ++g) {
          if (g * GR < nr) {
            T s0 = (T)0, s1 = (T)0;
#pragma unroll
            for (int u = 0; u < GR; ++u) {
              const int t = g * GR + u;
              const T rowv = sh.rowsh[wave][t] + shift;
              T rs = (T)0;
#pragma unroll
              for (int c = 0; c < NCOL; ++c) {
                const T tt = rowv + colv[c] - pc[t][c];
                const T tp = relu_of(tt);
                s1 += tp * tp;
                const T xn = relu_of(xr[t][c] + tt);
                xr[t][c] = xn;
                rs = c == 0 ? xn : rs + xn;
                cd[c] += (double)xn;
                s0 += pc[t][c] * xn;
              }
              sh.rowp[wave][t][lane] = rs;
            }
            s0d += (double)s0;
            s1d += (double)s1;
          }
        }
#pragma unroll
        for (int c = 0; c < NCOL; ++c) sh.colp[wave][lane + kWave * c] = cd[c];
        if (!replay) sh.mon0[k & 1][wave][lane] = fold32(s0d, s1d);
      }
      small_barrier();
      if (!replay && __builtin_amdgcn_readfirstlane(sh.stop) > 0) {
        stopped = true;  // iteration k was the last one
        break;
      }

      // Row sums: lanes 4 r .. 4 r + 3 a quarter of row r each, starting at
      // different chunks so that the lanes read different banks.
      double r2 = 0.0, pphi = 0.0, r1 = 0.0;
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        if (16 * p < nr) {
          const int r = 16 * p + (lane >> 2);
          const T* const src = &sh.rowp[wave][r < RT ? r : 0][(lane & 3) * 16];
          const int turn = sizeof(T) == 4 ? lane >> 1 : lane;
          double u[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            T v[VEC];
            load_chunk<T, VEC, false>(src + ((q + turn) & (Q - 1)) * VEC, v);
#pragma unroll
            for (int e = 0; e < VEC; ++e) u[(q * VEC + e) & 3] += (double)v[e];
          }
          double usum = (u[0] + u[1]) + (u[2] + u[3]);
          usum += dpp<0xB1>(usum);
          usum += dpp<0x4E>(usum);
          const double pm = (double)marg[p];
          const double res = usum - pm;
          const double ph = div_by(ra[p] - 2.0 * res, dn, in);
          ra[p] -= res;
          rph[p] = ph;
          if ((lane & 3) == 0 && r < nr) {
            sh.rowsh[wave][r] = (T)ph;
            r2 += res * res;
            pphi += pm * ph;
            r1 += res;
          }
        }
      }
      if (!replay) sh.mon1[wave][lane] = fold32(r2, pphi);
      if (SmallShared<T, NCOL>::NR > 0 && (lane & 3) == 0) sh.rsum[wave * (kWave / 4) + lane / 4] = r1;
      ++k;
      if (!replay && k % kSmallSnap == 0 && k < limit) {
        save();
        base_k = k;
      }
      small_barrier();
    }
    if (!stopped) {
      save();
      return;
    }
    limit = k;
    replay = true;
  }
}

// Wave 11.
template <typename T, int NCOL>
__device__ __forceinline__ void small_service(SmallShared<T, NCOL>& sh, const SweepArgs& a,
                                              const StateIn& sv, const T rhoT, int limit) {
  constexpr int NW = kSmallWaves, NR = SmallShared<T, NCOL>::NR;
  const int lane = threadIdx.x & (kWave - 1);
  const int n = (int)a.g.n;
  const double dm = (double)a.g.m, dn = (double)n, dmn = (double)a.g.m + (double)n;
  const double im = 1.0 / dm, in = 1.0 / dn, imn = 1.0 / dmn, irho = 1.0 / (double)rhoT;
  double cb[NCOL], cps[NCOL], marg[NCOL];  // b, psi~, q
  double cphi = sv.cphi, cpsi = sv.cpsi, alpha = sv.alpha;
  double base[3] = {cphi, cpsi, alpha};  // of the state in memory
#pragma unroll
  for (int c = 0; c < NCOL; ++c) {
    const int j = lane + kWave * c;
    marg[c] = j < n ? (double)static_cast<const T*>(a.q)[j] : 0.0;
  }
  // sum q - sum p: sum r is sum s + qp, and both are small numbers.
  double qp = 0.0;
#pragma unroll
  for (int c = 0; c < NCOL; ++c) qp += marg[c];
  for (int i = lane; i < (int)a.g.m; i += kWave) qp -= (double)static_cast<const T*>(a.p)[i];
  qp = wave_sum(qp);
  ScalarStep f;  // the latest tested iteration
  f.done = 0;
  f.status = 0;
  if (lane == 0) sh.stop = 0;
  // Float64 with few columns: alpha as with beta from sum r, which is there an
  // iteration's end later.  Few columns' sums have larger rounding errors than many
  // rows', and alpha would gather them: nu of 256 x 3 was 2.6 times as far from the
  // exact iterate after 1000 iterations, of 256 x 10 1.2 times, and no further from
  // 4 n = m on, where the sum would take 0.1 us more of 1.6 at 31 x 31.
  const bool tall = NR > 0 && 4 * (int64_t)n <= a.g.m;
  if (NR > 0 && lane >= NW * (kWave / 4) - (NR - 1) * kWave) sh.rsum[(NR - 1) * kWave + lane] = 0.0;
  auto save = [&]() {
#pragma unroll
    for (int c = 0; c < NCOL; ++c) {
      const int j = lane + kWave * c;
      if (j < n) {
        a.b[j] = cb[c];
        a.psi64[j] = cps[c];
        static_cast<T*>(a.psiT)[j] = (T)cps[c];
      }
    }
  };

  int base_k = 0, k = 0;
  bool replay = false;
  for (;;) {
    k = base_k;
    cphi = base[0];
    cpsi = base[1];
    alpha = base[2];
#pragma unroll
    for (int c = 0; c < NCOL; ++c) {
      const int j = lane + kWave * c;
      cb[c] = j < n ? a.b[j] : 0.0;
      cps[c] = j < n ? a.psi64[j] : 0.0;
      sh.colsh[j] = j < n ? static_cast<const T*>(a.psiT)[j] : (T)0;
    }
    if (lane == 0) sh.shift = (T)(cphi + cpsi);
    small_barrier();

    bool stopped = false;
    while (k < limit) {
      small_barrier();
      if (!replay && f.done) {
        stopped = true;
        break;
      }
      // s = column sums - q, their total, and steps 5-8.
      __builtin_amdgcn_s_setprio(3);
      double s[NCOL], tot = 0.0;
#pragma unroll
      for (int c = 0; c < NCOL; ++c) {
        double v[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) v[w] = sh.colp[w][lane + kWave * c];
        s[c] = (((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]))) +
               ((v[8] + v[9]) + v[10]) - marg[c];
        tot += s[c];
        if (c % 2 == 1) __builtin_amdgcn_sched_barrier(0);  // 22 values in flight are enough
      }
      tot = wave_sum(tot) + qp;
      const double beta = div_by(tot, dmn, imn);
      const double cc = 2.0 * beta - alpha;
      cphi = div_by(cc, dn, in);
      cpsi = div_by(cc, dm, im);
      alpha -= beta;
      if (lane == 0) sh.shift = (T)(cphi + cpsi);
      double s2 = 0.0, qpsi = 0.0;  // nothing beyond column n: s, q and b are 0 there
#pragma unroll
      for (int c = 0; c < NCOL; ++c) {
        const double ps = div_by(cb[c] - 2.0 * s[c], dm, im);
        cb[c] -= s[c];
        cps[c] = ps;
        sh.colsh[lane + kWave * c] = (T)ps;
        s2 += s[c] * s[c];
        qpsi += marg[c] * ps;
      }
      __builtin_amdgcn_s_setprio(0);
      ++k;
      if (!replay && k % kSmallSnap == 0 && k < limit) {
        save();
        base[0] = cphi;
        base[1] = cpsi;
        base[2] = alpha;
        base_k = k;
      }
      small_barrier();

      if (tall) {
        double r1 = 0.0;
#pragma unroll
        for (int i = 0; i < NR; ++i) r1 += sh.rsum[lane + kWave * i];
        alpha -= (wave_sum(r1) - tot) * imn;
        if (base_k == k) base[2] = alpha;
      }

      // The stopping test of iteration k, while the others sweep.
      if (!replay) {
        double v[3] = {0.0, 0.0, fold32(s2, qpsi)};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          v[0] += sh.mon0[(k - 1) & 1][w][lane];
          v[1] += sh.mon1[w][lane];
        }
        v[0] *= lane < 32 ? irho : 1.0;  // <rho C,X> to <C,X>
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q] += dpp<0xB1>(v[q]);
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q] += dpp<0x4E>(v[q]);
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q] += dpp<0x141>(v[q]);
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q] += dpp<0x140>(v[q]);
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q] += dpp<0x142, 0xA>(v[q]);
        const double ws[8] = {0.0, read_lane(v[1], 31), read_lane(v[1], 63), 0.0,
                              read_lane(v[2], 31), read_lane(v[2], 63),
                              read_lane(v[0], 31), read_lane(v[0], 63)};
        f.cphi = cphi;
        f.cpsi = cpsi;
        f.alpha = alpha;
        f.k = sv.iter + k;
        scalar_tests(f, sv, ws, false);
        if (lane == 0) {
          const int64_t slot = f.k - 1 < a.trace_cap ? f.k - 1 : (f.k - 1) % a.trace_cap;
          trace_record(a.trace + slot * kTraceWidth, f, sv.t_start, wall_clock64(), a.wall_rate);
          if (f.done) sh.stop = k;
        }
      }
    }
    if (!stopped) break;
    limit = k;
    replay = true;
  }
  save();
  if (lane == 0) {
    DevState* const st = a.st;
    const uint64_t now = wall_clock64();
    st->alpha = alpha;
    st->cphi = cphi;
    st->cpsi = cpsi;
    st->iter = sv.iter + k;
    st->t_last = now;
    st->pobj = f.pobj;
    st->dobj = f.dobj;
    st->rp = f.rp;
    st->rd = f.rd;
    st->gap = f.gap;
    st->test = f.test;
    if (f.done) {
      st->done = 1;
      st->status = f.status;
      st->stop_iter = f.k;
      st->t_stop = now;
    }
  }
}

template <typename T, int NCOL>
__global__ __launch_bounds__(kSmallBlock) void small_kernel(SweepArgs a, int64_t iters) {
  __shared__ __align__(16) SmallShared<T, NCOL> sh;
  const StateIn sv = load_state(a.st);
  if (sv.done) return;
  const int64_t left = sv.max_iter - sv.iter;
  const int limit = (int)(iters < left ? iters : left);
  if (limit <= 0) return;
  const T rhoT = (T)sv.rho;
  if (__builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave) == kSmallWaves)
    small_service<T, NCOL>(sh, a, sv, rhoT, limit);
  else
    small_sweep<T, NCOL>(sh, a, rhoT, limit);
}

}  // namespace
}  // namespace drot
